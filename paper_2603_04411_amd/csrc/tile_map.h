// XCD-aware workgroup -> tile mapping (shared by the MFMA kernels; also compiled on the host
// by the unit test of the mapping).
#pragma once

#include <stdint.h>

#ifdef LMHEAD_TILE_MAP_HOST
#define LMHEAD_HD
#else
#include <hip/hip_runtime.h>
#define LMHEAD_HD __host__ __device__
#endif

namespace lmhead {

// Workgroup -> tile mapping that keeps L2 traffic local to an XCD.
//
// The chip dispatches workgroup i of a 1-D grid to XCD i % 8, and each XCD has a private L2.
// A work grid of X x Y items (x selects the A-side operand slab, y the B-side slab) is shared out so
// that every XCD gets the same number of items, give or take one:
//  - the first 8 floor(Y / 8) values of y in eight contiguous ranges, one per XCD.  Inside its range an XCD
//    walks blocks of bx x by items (x fastest), so the 32 workgroups it runs at a time cover a compact block and
//    share bx + by operand slabs instead of fetching 64;
//  - the items of the remaining r = Y % 8 values of y in eight contiguous pieces of the order "y fastest, then x":
//    neighbours share the x slab, and all of them the r slabs of y.
// (Cutting Y into eight ranges of ceil(Y / 8) leaves XCDs idle when Y is small: at 41 token blocks one of the
// eight has nothing to do, at one token block seven.  Forward of 120 tokens x 151936: 838 -> 182 us; the 8x8x256
// step, 41 blocks: 19.2 -> 18.4 ms; 160 blocks or more: no change.)
// Returns false for workgroups beyond the work (the grid is sized for the largest possible Y).
constexpr int kNumXcd = 8;
LMHEAD_HD inline bool xcd_tile_coords(int wg, int X, int Y, int bx, int by, int& x, int& y) {
  const int xcd = wg % kNumXcd;
  const int j = wg / kNumXcd;
  const int y_per = Y / kNumXcd;
  if (j >= y_per * X) {
    const int rest = Y - y_per * kNumXcd;
    const int64_t items = (int64_t)rest * X;
    const int i = (int)(items * xcd / kNumXcd) + (j - y_per * X);
    if (i >= (int)(items * (xcd + 1) / kNumXcd)) return false;
    x = i / rest;
    y = y_per * kNumXcd + (i - x * rest);
    return true;
  }
  const int per_yblk = X * by;
  const int yb = j / per_yblk;
  int r = j - yb * per_yblk;
  const int h = min(by, y_per - yb * by);
  const int nfull = X / bx;
  const int full_items = nfull * bx * h;
  int yin;
  if (r < full_items) {
    const int xb = r / (bx * h);
    const int r2 = r - xb * (bx * h);
    yin = r2 / bx;
    x = xb * bx + (r2 - yin * bx);
  } else {
    const int tw = X - nfull * bx;
    r -= full_items;
    yin = r / tw;
    x = nfull * bx + (r - yin * tw);
  }
  y = xcd * y_per + yb * by + yin;
  return true;
}
// Grid size that covers every item for any Y <= Y_cap under the mapping above (an XCD's share grows with Y and
// does not depend on the block shape).
inline unsigned xcd_grid_size(int X, long long Y_cap, int /*by*/) {
  const long long rest = Y_cap % kNumXcd;
  return (unsigned)(kNumXcd * (Y_cap / kNumXcd * X + (rest * X + kNumXcd - 1) / kNumXcd));
}

// Relative rate of the 256, 128 and 64 wide tiles once the chip is full: 65536 x 1024 x 1024 in bf16 takes 143, 179 and
// 252 us, in fp32 (a quarter of the tokens) 254, 254 and 269.
inline float tile_rate(int edge, bool f32) {
  return edge == 256 ? 1.f : edge == 128 ? (f32 ? 1.f : 0.8f) : (f32 ? 0.95f : 0.57f);
}

// Compute units that the launch rules count on (a GPU need not be present where workspaces are sized).
constexpr int kComputeUnits = 256;

// Slices of dH's contraction over the vocabulary: a tile grid that fills the chip's rounds badly (few tokens, or
// 1.4 rounds of tiles) is cut into `ks` slices per tile, summed in order afterwards.  The number of tiles follows from
// N_v, which only the device knows, so the index kernel picks ks there (WsHeader::ksplit): the cheapest allowed one,
// the fewest slices on a tie.  (Picked on the host from the capacity, 20 token blocks x 16 tiles along d of a step with
// room for 32 blocks took three slices and 5.43 ms; now four and 4.89.)
constexpr int kSplitTiles = 2048, kMaxSplit = 64;
struct DhSplit {
  int m_tiles;   // tiles along d
  int edge;
  int ksteps;    // K-steps of a vocabulary chunk
};
// Time of a split in K-steps of a 256 wide tile: rounds of workgroups, each a slice's K-steps plus about ten for its
// pipeline fill and epilogue; then the sum, 512 KB per 256 x 256 slice tile at memory speed (0.085) and a launch.
LMHEAD_HD inline float dh_split_cost(const DhSplit& p, int n_tiles, int ks) {
  const int tiles = p.m_tiles * n_tiles;
  const int rounds = (tiles * ks + kComputeUnits - 1) / kComputeUnits;
  const int steps = (p.ksteps + ks - 1) / ks;
  const float area = (float)p.edge / 256.f;
  return (float)rounds * (float)(steps + 10) + (ks > 1 ? 8.f + 0.085f * area * (float)(tiles * ks) : 0.f);
}
// At most kSplitTiles slice tiles exist when there are several per tile, which bounds the scratch.
LMHEAD_HD inline bool dh_split_allowed(const DhSplit& p, int n_tiles, int ks) {
  return ks == 1 || ((int64_t)p.m_tiles * n_tiles * ks <= kSplitTiles && ks <= p.ksteps);
}
// Slice tiles that scratch is needed for at any number of tokens up to n_tiles tiles of them (single: also when ks = 1).
inline int64_t dh_split_tiles(const DhSplit& p, int64_t n_tiles, bool single) {
  const int64_t tiles = p.m_tiles * n_tiles;
  const int64_t split = tiles * kMaxSplit < kSplitTiles ? tiles * kMaxSplit : kSplitTiles;
  return single && split < tiles ? tiles : split;
}

}  // namespace lmhead
