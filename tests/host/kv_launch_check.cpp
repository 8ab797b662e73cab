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
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
