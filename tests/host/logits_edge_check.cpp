// Host check of the rule that picks the logits kernels' tile edge: it widens with the number of slots, and the scratch for the
// per-tile statistics at n slots holds what any smaller number of slots needs.
#include <algorithm>
#include <cstdio>
using std::min;
#define LMHEAD_TILE_MAP_HOST 1
#include "../../paper_2603_04411_amd/csrc/tile_map.h"

int main() {
  using namespace lmhead;
  long bad = 0, cases = 0;
  for (bool f32 : {false, true})
    for (int64_t V : {1, 63, 64, 65, 100, 4096, 8000, 16384, 32768, 50257, 151936, 300000, 4000000}) {
      int edge = 0;
      int64_t scratch = 0;
      for (int64_t n = 1; n < 200000; n += n < 2000 ? 1 : n / 300) {
        ++cases;
        const int e = logits_edge(f32, V, n);
        if (e < edge || (e != 64 && e != 128 && e != 256)) ++bad;
        edge = e;
        const int64_t part = logits_part_slots(f32, V, n);
        const int64_t need = (V + e - 1) / e * ((n + kTile - 1) / kTile * kTile);
        if (part < need || part < scratch) ++bad;
        scratch = part;
      }
    }
  // over a large vocabulary the number of slots decides: one tile of 64, one of 128 at a share of 5/8 valid, 256 beyond
  for (int64_t V : {50257, 151936}) {
    const int64_t n[] = {1, 64, 65, 128, 200, 204, 205, 256, 4096};
    const int want[] = {64, 64, 128, 128, 128, 128, 256, 256, 256};
    for (int i = 0; i < 9; ++i, ++cases)
      if (logits_edge(false, V, n[i]) != want[i]) ++bad;
  }
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
