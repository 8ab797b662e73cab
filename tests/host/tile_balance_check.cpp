// Host check that the XCD-aware tile walk gives every XCD the same number of items, give or take one, and that its
// grid holds no more than the workgroups that needs.
#include <algorithm>
#include <cstdio>
using std::min;
#define LMHEAD_TILE_MAP_HOST 1
#include "../../paper_2603_04411_amd/csrc/tile_map.h"

int main() {
  long bad = 0, cases = 0;
  for (int X : {1, 3, 8, 16, 594, 1188})
    for (int Y : {1, 2, 7, 8, 9, 15, 26, 41, 64, 161}) {
      ++cases;
      const unsigned g = lmhead::xcd_grid_size(X, Y, 4);
      int per[lmhead::kNumXcd] = {};
      for (unsigned wg = 0; wg < g; ++wg) {
        int x, y;
        if (lmhead::xcd_tile_coords((int)wg, X, Y, 4, 4, x, y)) per[wg % lmhead::kNumXcd]++;
      }
      const int lo = *std::min_element(per, per + lmhead::kNumXcd), hi = *std::max_element(per, per + lmhead::kNumXcd);
      if (hi - lo > 1 || (long)g != 8l * hi) ++bad;
    }
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
