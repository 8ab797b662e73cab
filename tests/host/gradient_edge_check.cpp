// Host check of the rules that pick the tile edges of dH and dW, at sizes where another edge was measured to be 10 % slower or
// more: contractions that are long enough for wide tiles' rate to count take them, short ones narrow tiles.
#include <algorithm>
#include <cstdio>
using std::min;
#define LMHEAD_TILE_MAP_HOST 1
#include "../../paper_2603_04411_amd/csrc/tile_map.h"

int main() {
  using namespace lmhead;
  long bad = 0, cases = 0;
  auto dh = [&](bool f32, int d, int n, int V, int want) {
    ++cases;
    const int64_t ksteps = (int64_t)(V + 255) / 256 * 256 * (f32 ? 4 : 2) / 128;
    if (dh_edge(f32, d, n, ksteps) != want) { ++bad; std::printf("dH f32=%d d=%d n=%d V=%d: %d\n", f32, d, n, V, dh_edge(f32, d, n, ksteps)); }
  };
  for (int n : {2048, 4096, 8192}) {
    dh(true, 1024, n, 32000, 256);
    dh(true, 1024, n, 16000, 256);
    dh(true, 512, n, 20000, 256);
  }
  dh(true, 1024, 512, 32000, 128);
  dh(true, 256, 1024, 30000, 128);
  dh(true, 256, 256, 4096, 64);
  dh(true, 1024, 64, 32000, 64);
  dh(true, 1024, 6000, 500, 64);
  dh(false, 4096, 4096, 32000, 256);
  dh(false, 256, 256, 4096, 64);
  auto dw = [&](bool f32, int d, int V, int n, int want) {
    ++cases;
    const int got = dw_edge(f32, d, V, n);
    if (got != want) { ++bad; std::printf("dW f32=%d d=%d V=%d n=%d: %d\n", f32, d, V, n, got); }
  };
  // full rounds of 256 wide tiles, a few tiles whose contraction can be cut, tiles that do not divide a round
  for (int n : {4096, 16384}) {
    dw(false, 1024, 16384, n, 256);
    dw(false, 1024, 32768, n, 256);
    dw(false, 2048, 16384, n, 256);
    dw(false, 4096, 8192, n, 256);
    dw(false, 512, 32768, n, 256);
    dw(false, 5120, 6000, n, 256);
    dw(false, 1024, 20000, n, 256);
    dw(false, 2048, 12000, n, 256);
  }
  for (int d : {512, 1024, 2048, 4096}) dw(false, d, 2048 * 1024 / d, 16384, 256);
  dw(false, 2048, 5000, 16384, 256);
  dw(true, 1024, 32000, 8192, 256);
  dw(true, 512, 20000, 8192, 64);
  // a handful of tiles: their contraction cut into slices beats a few narrow tiles on a few compute units
  for (int d : {64, 256, 512, 1024}) dw(false, d, 300, 16000, 256);
  dw(false, 512, 300, 6000, 256);
  dw(false, 4096, 300, 6000, 64);
  dw(false, 1024, 2048, 8000, 64);
  // short contractions
  dw(false, 512, 300, 500, 64);
  dw(false, 1024, 151936, 300, 256);
  dw(false, 2048, 151936, 384, 256);
  dw(false, 1024, 20000, 1024, 128);
  dw(false, 2048, 12000, 1024, 128);
  dw(false, 1024, 40000, 256, 128);
  dw(false, 1024, 151936, 150, 128);
  dw(false, 4096, 151936, 192, 128);
  dw(false, 1024, 2048, 1024, 64);
  dw(false, 512, 4096, 256, 64);
  dw(true, 512, 4096, 1024, 64);
  dw(true, 1024, 32000, 256, 128);
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
