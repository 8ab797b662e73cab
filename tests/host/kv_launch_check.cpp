// Host check of the rules that merge launches of the KV path: the merged form is taken where it was measured to be the faster one.
#include <algorithm>
#include <cstdio>
using std::min;
#define LMHEAD_TILE_MAP_HOST 1
#include "../../paper_2603_04411_amd/csrc/tile_map.h"

int main() {
  using namespace lmhead;
  long bad = 0, cases = 0;
  // the mask in the launch of the logits, without soft outputs: bytes of a component, tokens, components
  auto mask = [&](int esz, int64_t n, int d, bool want) {
    ++cases;
    if (!kv_few_fits(esz == 4, n, d) || kv_mask_with_logits(esz, n, d, false) != want) { ++bad; std::printf("mask esz=%d n=%ld d=%d\n", esz, (long)n, d); }
  };
  for (int n : {1, 16, 64, 540, 2000}) mask(2, n, 256, true), mask(4, n, 256, true);
  mask(2, 8000, 64, true);
  for (int n : {1, 16, 256, 540}) mask(2, n, 448, true);
  mask(2, 1000, 448, false);
  for (int d : {640, 704, 768}) mask(2, 16, d, true), mask(2, 64, d, true);
  mask(2, 240, 640, false);
  mask(2, 200, 704, false);
  for (int d : {768, 832, 896, 960})
    for (int n : {128, 200, 300, 540}) mask(2, n, d, false);
  for (int n : {1, 16, 32}) mask(2, n, 1024, true);
  for (int n : {64, 128, 200}) mask(2, n, 1024, false);
  for (int n : {16, 64, 100}) mask(4, n, 448, true);
  for (int n : {160, 300, 1000}) mask(4, n, 448, false);
  for (int d : {640, 704, 768, 832, 896, 960, 1024})
    for (int n : {16, 200, 300}) mask(4, n, d, false);
  mask(2, 16, 1088, false);
  // what follows g_x~ in a backward call: one launch or several, dx within it or not
  auto tail = [&](bool f32, int64_t n, int d, bool one, bool apart) {
    ++cases;
    const KvTail t = kv_tail(f32, n, d, kv_gradient_slices(f32, n, d));
    if ((t.edge != 0) != one || (one && kv_tail_dx_apart(f32, n, d, t) != apart)) { ++bad; std::printf("tail f32=%d n=%ld d=%d\n", f32, (long)n, d); }
  };
  const struct { int64_t n; int d; bool one, apart; } bf16[] = {
      {64, 64, true, false}, {700, 256, true, false}, {2000, 512, true, false}, {32768, 256, true, false}, {16384, 384, true, false},
      {14000, 640, true, false}, {4096, 1024, true, false}, {1500, 1536, true, false}, {2048, 2048, true, false}, {3000, 2048, false, false},
      {65536, 64, false, false}, {16384, 448, false, false}, {32768, 448, false, false}, {32768, 384, false, false}, {40000, 320, false, false},
      {16, 1024, true, false}, {16, 4096, true, true}, {256, 2560, true, false}, {100, 3072, true, true}, {256, 4096, true, true},
      {300, 4096, true, false}, {100, 5120, true, true}, {60, 6144, true, true}, {100, 8192, true, true}};
  for (const auto& c : bf16) tail(false, c.n, c.d, c.one, c.apart);
  const struct { int64_t n; int d; bool one, apart; } fp32[] = {
      {100, 64, true, true}, {300, 128, true, true}, {40, 192, true, true}, {100, 256, true, true}, {300, 192, false, false}, {300, 256, false, false},
      {512, 320, false, false}, {16, 512, false, false}, {100, 448, false, false}, {16, 640, false, false}, {16, 768, false, false},
      {1500, 448, true, false}, {2000, 576, true, false}, {1000, 768, true, false}, {300, 1024, true, true}, {600, 1280, true, false},
      {1000, 1152, true, false}, {800, 1280, true, false}, {1200, 896, true, false}, {400, 1792, true, false}, {800, 960, true, true},
      {600, 1408, true, true}, {400, 1536, true, true}, {256, 2560, true, true}, {2000, 256, false, false}, {4096, 1024, false, false}};
  for (const auto& c : fp32) tail(true, c.n, c.d, c.one, c.apart);
  // the scratch is sized for the slices of launches of their own, and one counter per tile of both gradients on edge 64
  for (bool f32 : {false, true})
    for (int d = 64; d <= 8192; d += d < 2048 ? 64 : 320)
      for (int64_t n = 1; n < 200000; n += n < 600 ? 7 : n / 40) {
        ++cases;
        const KvTail own = kv_gradient_slices(f32, n, d), t = kv_tail(f32, n, d, own);
        if (own.slices < 1 || (own.edge != 64 && own.edge != 128 && own.edge != 256)) ++bad;
        if (!t.edge) continue;
        if ((t.edge != 64 && (f32 || t.edge != 128)) || t.slices < 1 || t.slices > own.slices || (f32 && t.slices != own.slices)) ++bad;
        if (2 * tiles_of(d, d, t.edge) > kv_tail_counters(d)) ++bad;
      }
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
