// Host check of the rule that picks the logits kernels' tile edge: it widens with the number of slots, and the scratch for the
// per-tile statistics at n slots holds what any smaller number of slots needs, in tiles or in ranges of the vocabulary; and the forward
// takes ranges where they were measured to be the faster ones.  With arguments (V d n, repeated) it prints 1 for ranges, 0 for tiles.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
using std::min;
#define LMHEAD_TILE_MAP_HOST 1
#include "../../paper_2603_04411_amd/csrc/tile_map.h"

int main(int argc, char** argv) {
  using namespace lmhead;
  if (argc > 1) {
    for (int i = 1; i + 2 < argc; i += 3) std::printf("%d\n", (int)logits_stream(std::atoll(argv[i]), std::atoll(argv[i + 1]), std::atoll(argv[i + 2])));
    return 0;
  }
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
        const int64_t slots = (n + kTile - 1) / kTile * kTile;
        int64_t need = (V + e - 1) / e * slots;
        if (!f32 && logits_stream(V, 1 << 20, n) && kComputeUnits * slots > need) need = kComputeUnits * slots;   // of any d
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
  // ranges or tiles: V, d and whether ranges are faster, by a step and by calls of the forward one after the other
  const struct { int64_t V, d; bool ranges; } w[] = {{32000, 2048, false}, {16384, 4096, false}, {30000, 4096, false}, {64000, 1024, false}, {151936, 512, false},
                                                     {60000, 2048, false}, {66000, 2048, false}, {132000, 1024, false}, {16400, 8192, false}, {18500, 8192, false},
                                                     {80000, 2048, true}, {100000, 2048, true}, {151936, 2048, true}, {151936, 1024, true},
                                                     {50000, 4096, true}, {20000, 8192, true}, {40000, 5120, true}, {2400000, 64, true}};
  for (const auto& c : w)
    for (int n : {1, 64, 192, 204}) {
      ++cases;
      if (logits_stream(c.V, c.d, n) != c.ranges || logits_stream(c.V, c.d, 205)) { ++bad; std::printf("V=%ld d=%ld n=%d\n", (long)c.V, (long)c.d, n); }
    }
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
