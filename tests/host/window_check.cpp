// Host check of the buffer windows through which the gate reads x, whatever its row pitch: dU, which takes x in pieces beyond one
// window, gets pieces of at least one K-step, so that the loop over them ends; the rows of a token tile of x U lie inside one.  And
// of W, which dH reads through them: no K-step starts behind it.
#include <algorithm>
#include <cstdio>
using std::min;
#define LMHEAD_TILE_MAP_HOST 1
#include "../../paper_2603_04411_amd/csrc/tile_map.h"

int main() {
  using namespace lmhead;
  long bad = 0, cases = 0;
  for (int esz : {2, 4})
    for (int d : {64, 1024, 8192})
      for (int64_t ldx = d; ldx > 0 && ldx < (int64_t)1 << 60; ldx += ldx / 97 / 8 * 8 + 8) {
        ++cases;
        const int64_t pitch = kv_gradient_needs_dense(ldx) ? d : ldx;
        const int64_t step = 128 / esz * (pitch * esz);
        const int piece = window_ksteps(step);
        if (piece < 1 || piece * step > kWindowBytes || pitch > longest_pitch(1)) { ++bad; continue; }
        int turns = 0;
        for (int k = 0; k < 64; k += piece) ++turns;
        if (turns > 64) ++bad;
      }
  // the rows of a token tile of x~ = x U, as its offsets address them, end inside a window; a copy is made only where they do not
  for (int esz : {2, 4})
    for (int d : {64, 1024, 8192})
      for (int edge : {64, 128, 256})
        for (int64_t n : {1, 2, 63, 64, 65, 300, 100000})
          for (int64_t ldx = d; ldx < (int64_t)1 << 32; ldx += ldx / 97 / 8 * 8 + 8) {
            ++cases;
            const int64_t pitch = kv_tiles_need_dense(n, edge, ldx, d, esz) ? d : ldx;
            if ((min(n, (int64_t)edge) - 1) * pitch * esz + d * esz > kWindowBytes) ++bad;
            if (pitch == d && ldx > d && (min(n, (int64_t)edge) - 1) * ldx * esz + d * esz <= kWindowBytes) ++bad;
          }
  // dH: every K-step of a vocabulary chunk, 64 or 32 rows of W, starts inside W
  for (int rows : {32, 64})
    for (int64_t V = 1; V < 20000; V += 1 + V / 50)
      for (int64_t tiles : {1, 4, 1024})
        for (int64_t c0 = 0; c0 < V; c0 += tiles * kTile) {
          ++cases;
          const int64_t left = (V - c0 + kTile - 1) / kTile, K = chunk_rows(V, c0, left < tiles ? left : tiles);
          const int64_t ksteps = (K + rows - 1) / rows;
          if (K < 1 || c0 + (ksteps - 1) * rows >= V || c0 + ksteps * rows < min(V, c0 + tiles * kTile)) ++bad;
        }
  // the strides around the line, and the first that one K-step does not fit
  for (int64_t ldx : {(int64_t)64, (int64_t)1 << 20, (int64_t)1 << 22, ((int64_t)1 << 23) - 8})
    if (++cases, kv_gradient_needs_dense(ldx)) ++bad;
  for (int64_t ldx : {(int64_t)1 << 23, ((int64_t)1 << 24) - 8, (int64_t)1 << 24, (int64_t)1 << 26, (int64_t)1 << 40})
    if (++cases, !kv_gradient_needs_dense(ldx)) ++bad;
  if (window_ksteps(128 * ((int64_t)1 << 24)) != 0) ++bad;
  std::printf("cases=%ld bad=%ld\n", cases, bad);
  return bad != 0;
}
