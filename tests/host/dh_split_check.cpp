// Host check of the rule that cuts dH's contraction into slices: for any number of token tiles up to the capacity, the
// slices it may pick fit the scratch reserved for that capacity, one slice is always allowed, and a grid that
// already fills the chip's rounds is left whole.
#include <algorithm>
#include <cstdio>
using std::min;
#define LMHEAD_TILE_MAP_HOST 1
#include "../../paper_2603_04411_amd/csrc/tile_map.h"

int main() {
  using namespace lmhead;
  long bad = 0, cases = 0;
  for (int m : {1, 2, 4, 14, 16, 20, 128, 3000})
    for (int edge : {64, 128, 256})
      for (int ksteps : {1, 2, 8, 128, 594 * 4})
        for (int cap : {1, 2, 5, 41, 128, 2048}) {
          const DhSplit p{m, edge, ksteps};
          for (int n = 0; n <= cap; n = n < 8 ? n + 1 : n * 3 / 2) {
            ++cases;
            int ks = 0;
            for (int q = 1; q <= kMaxSplit; ++q)
              if (dh_split_allowed(p, n, q) && (ks == 0 || dh_split_cost(p, n, q) < dh_split_cost(p, n, ks))) ks = q;
            if (ks < 1 || ks > ksteps) ++bad;
            const long long tiles = (long long)m * n;
            if (ks > 1 && tiles * ks > dh_split_tiles(p, cap, false)) ++bad;
            if (tiles * ks > dh_split_tiles(p, cap, true) && n > 0) ++bad;
            if (tiles % kComputeUnits == 0 && tiles > 0 && ks != 1) ++bad;
          }
        }
  // 8 tiles of 2376 K-steps fill the chip 32 times over
  const DhSplit few{8, 256, 2376};
  int ks = 1;
  for (int q = 1; q <= kMaxSplit; ++q)
    if (dh_split_allowed(few, 1, q) && dh_split_cost(few, 1, q) < dh_split_cost(few, 1, ks)) ks = q;
  if (ks != 32) ++bad;
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
