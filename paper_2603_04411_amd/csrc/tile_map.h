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

// Macro-tile of the contractions: the widest tile edge, and the unit that operands are padded to.
constexpr int kTile = 256;

// Vocabulary rows of a chunk of n_tiles tiles from row c0 on.  Both gradients end there: dH's contraction has no K-step that starts
// behind W, where a buffer window (whose range check subtracts the K-step's offset from its size) promises nothing.
inline int64_t chunk_rows(int64_t V, int64_t c0, int64_t n_tiles) { return V - c0 < n_tiles * kTile ? V - c0 : n_tiles * kTile; }

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

// Most bytes that a buffer descriptor covers, and the K-steps of a K-major operand, `step` bytes apart, inside them: a longer
// contraction is taken in pieces of that many.
constexpr int64_t kWindowBytes = 0x7fffffff;
LMHEAD_HD inline int window_ksteps(int64_t step) { return (int)(kWindowBytes / step); }
// A K-step of a K-major operand is 128 times its row pitch in elements (64 rows in bf16, 32 in fp32): the longest pitch that leaves
// room for `ksteps` of them.
constexpr int64_t longest_pitch(int ksteps) { return kWindowBytes / (128 * ksteps); }
// dU reads x where it lies while a window holds this many K-steps, and a dense copy of it beyond.  Backward call, bf16, us, where it
// lies / copied, at 7, 3 and 1 K-steps a window: 1024 x 1024 48.8 / 48.6   50.2 / 48.6   56.0 / 48.8;   4096 x 1024 92.6 / 96.2
// 94.9 / 95.6   102.1 / 95.6;   16384 x 1024 at 15 and 3: 255 / 254   261 / 257.
constexpr int kLeastPiece = 2;
inline bool kv_gradient_needs_dense(int64_t ldx) { return ldx > longest_pitch(kLeastPiece); }
// The tiled projection addresses the rows of a token tile through one window: x is copied where they do not fit.
inline bool kv_tiles_need_dense(int64_t n, int edge, int64_t ldx, int d, int esz) {
  const int64_t rows = n < edge ? n : edge;
  return rows > 1 && ldx > (kWindowBytes / esz - d) / (rows - 1);
}

// Compute units that the launch rules count on (a GPU need not be present where workspaces are sized).
constexpr int kComputeUnits = 256;

// Tile edges of the LM-head kernels (four wavefronts per tile whatever the edge; 256 / edge workgroups share a compute
// unit).  256 needs the fewest operand bytes per flop, the only edge the vector L1 feeds at full bf16 rate.  The smaller
// ones give more and shorter tiles when 256 x 256 would leave most of the chip idle, waste less on padding when
// there are few tokens, and two or four workgroups on a compute unit overlap one's stores with another's loads.
inline int64_t tiles_of(int64_t m, int64_t n, int edge) { return ((m + edge - 1) / edge) * ((n + edge - 1) / edge); }
// Logits (forward and dZ): V = vocabulary rows, n = token slots.  A pass over several weight matrices takes the edge of a
// single one: the edge groups the terms of the softmax, and the two calls promise the same bits.
// The most slots that a call may have for its tiles to be `edge` wide or narrower.  Either one round of tiles, two to a
// compute unit (fp32, edge 64: up to four rounds of 256 wide tiles, matrix-core bound on any edge, so that narrow tiles only
// even out the rounds).  Or so few tokens that one tile holds them all and narrower ones are padded less: 64 wide up to
// 64 slots; 128 wide while 5/8 of the slots fit, the share that is valid where lengths are uniform in [T/4, T].  N_v is not
// known here: over 128 valid tokens 256 wide tiles win where W is long and wide, below that 128 wide ones, by as much.
// Forward + dZ, us, edge 256 / 128 / 64 (V 151936 unless said):
//   slots (valid)   64 (64)          128 (128)        200 (120)        200 (200)        256 (256)        320 (192)
//   d 2048          480/400/354      479/405/412      473/405/412      472/462/634      474/461/640      470/470/512
//   d 4096          713/624/574      715/625/747      707/618/746      711/812/1203     716/813/1219     708/808/958
//   d 4096 V 32000  235/171/176      239/175/218      234/175/218      239/214/312      240/214/313      239/210/250
//   d 1024 V 32000  66/37/32         66/37/41         66/36/42         67/47/64         70/49/64         68/46/55
//   fp32, all valid: n 256 d 256 V 4096 155/49/25   n 1024 d 512 V 20000 538/335/339   n 4096 d 1024 V 16000 1982/1949/2076
inline int64_t logits_slots(bool f32, int64_t V, int edge) {
  const int64_t few = edge == 64 ? 64 : 128 * 8 / 5;
  int64_t n = 2 * kComputeUnits / ((V + edge - 1) / edge) * edge;
  if (f32 && edge == 64) {
    const int64_t four = 4 * kComputeUnits / ((V + kTile - 1) / kTile) * kTile;
    n = n > four ? n : four;
  }
  return n > few ? n : few;
}
inline int logits_edge(bool f32, int64_t V, int64_t n) {
  return n <= logits_slots(f32, V, 64) ? 64 : n <= logits_slots(f32, V, 128) ? 128 : kTile;
}
// The forward of as many bf16 slots as 128 wide tiles are for, over a W that the last-level cache (256 MB) cannot hold or mostly hold:
// one range of rows per compute unit instead of tiles (lmhead_stream.hip).  What is still there of a smaller W from the call before
// the tiles read sooner, and the ranges, which go past the caches, leave none of it to the dZ of a step.  Calls one after the other on
// the same W, us, tiles / ranges, 64 (64), 192 (120) and 200 (200) slots (valid); steps are forward, loss and backward:
//                           call                     step
//   below:  d 2048 V 32000  32/42   40/48   41/48      158/166 190/201 192/204
//           d 4096 V 16384  41/62   49/66   49/66      187/210 229/242 227/247
//           d 1024 V 64000  35/37   43/47   43/47      157/158 197/206 199/212
//           d 512 V 151936  43/44   60/63   59/63      181/188 259/267 268/282
//           d 2048 V 66000  65/71   85/100  87/101     354/355 468/438 486/461
//           d 4096 V 33000  69/68   93/117  95/119     349/346 472/453 494/483
//   above:  d 2048 V 80000  97/74   130/106 128/106    465/426 541/489 560/514
//           d 1024 V 151936 81/68   116/97  115/97     414/388 544/501 543/511
//           d 2048 V 151936 157/117 229/170 217/171    814/750 928/857 953/893
//           d 4096 V 50000  120/80  174/130 170/131    573/517 672/596 717/650
//           d 8192 V 20000  120/117 169/125 164/125    489/474 628/544 635/564
//           d 64 V 2100000  280/132 402/255 371/257
//           (fewer rows a range, most of whose tile is empty: d 8192 V 18500 112/116 167/125 167/124)
// (With other work in between, which takes W out of the caches, ranges are the faster ones for the smaller W too: d 2048 V 32000 68/50
// 85/55 79/55; but not for steps, 205/206 236/235 242/242, which read it twice.)
constexpr int64_t kStreamSlots = 128 * 8 / 5, kStreamBytes = (int64_t)288 << 20, kStreamRows = 76;
inline bool logits_stream(int64_t V, int64_t d, int64_t n) {
  return n <= kStreamSlots && V * d * 2 >= kStreamBytes && V >= kStreamRows * kComputeUnits;
}
// Per-tile softmax statistics (planes x slots) that the logits of any number of slots up to n need: fewer slots take narrower
// tiles, i.e. more planes, and a workspace sized for a large batch has to serve the smaller ones.
inline int64_t logits_part_slots(bool f32, int64_t V, int64_t n) {
  int64_t most = 0;
  for (int edge : {64, 128, kTile}) {
    const int64_t slots = edge == kTile ? n : logits_slots(f32, V, edge);
    const int64_t need = (V + edge - 1) / edge * (((slots < n ? slots : n) + kTile - 1) / kTile * kTile);
    most = need > most ? need : most;
  }
  if (!f32 && V >= kStreamRows * kComputeUnits) {   // the planes of logits_stream, one per range
    const int64_t need = (int64_t)kComputeUnits * (((kStreamSlots < n ? kStreamSlots : n) + kTile - 1) / kTile * kTile);
    most = need > most ? need : most;
  }
  return most;
}
// The vocabulary tiles of a chunk of dW that would start a mostly empty last round of 256 wide tiles are contracted in slices
// that fill it: how many (1: the last round is full enough, or the tiles along d do not divide a round).
constexpr int kDwTailSlices = 8;
inline int dw_tail_slices(int64_t m_tiles, int64_t n_tiles, int cus) {
  if (m_tiles > cus || cus % m_tiles != 0) return 1;
  const int64_t rest = n_tiles % (cus / m_tiles);
  const int64_t ks = rest > 0 ? cus / (rest * m_tiles) : 1;
  return (int)(ks < kDwTailSlices ? ks : kDwTailSlices);
}
// dW: m = d, rows = vocabulary rows of a chunk, n = token slots (the contraction).  A tile of each edge costs a pipeline fill
// and an epilogue and then so much per K-step: the wide ones have the better rate, the narrow ones the cheaper ends and the
// fuller rounds.  Every tile of an edge takes the same time, so the cost of each edge can be written down, in K-steps (128
// bytes of a row) of a full round of 256 wide tiles (1.3 us in bf16, 7.3 us in fp32), and the cheapest is taken: on average
// within 0.5 % (bf16, 217 sizes) and 0.3 % (fp32, 68 sizes) of the best edge.  dW alone, us, edge 256 / 128 / 64:
//   bf16  d 1024 V 16384  n 256   23.4 / 22.6 / 27.7    n 1024 39.2 / 42.4 / 54.7    n 16384 348 / 505 / 1233   256 tiles: one round
//         d 1024 V 20000  n 256   52.2 / 27.2 / 31.6    n 1024 79.6 / 53.2 / 65.5    n 16384 456 / 631 / 1594   316 tiles: cut into slices
//         d 1024 V 2048   n 256   32.5 / 10.5 / 9.0     n 4096 40.9 / 37.4 / 31.8    n 16384 73.6 / 151 / 130   32 tiles: cut into 8
//         d 512 V 300     n 500   20.9 / 11.5 / 9.0    n 6000 31 / 48 / 40    n 16000 49 / 116 / 93    4 tiles: cut into 8
//         d 1024 V 151936 n 128   174 / 156 / 191    n 300 209 / 242 / 250      n 512   248 / 289 / 356
//         d 4096 V 151936 n 192   665 / 601 / 691       n 384  834 / 821 / 1042      n 512   929 / 941 / 1250
//   fp32  d 512 V 4096    n 256   39 / 24 / 16          n 2048 92 / 124 / 73         n 8192  264 / 468 / 263
//         d 1024 V 8000   n 256   65 / 42 / 45          n 2048 268 / 240 / 255       n 8192  929 / 932 / 1038
struct TileCost {
  // K-steps of a full round of 256 wide tiles: fill and epilogue per round; a K-step of a full round; a K-step of a tile that
  // has its compute unit for itself, its operands in L2 or beyond
  float ends, step, near, far;
};
inline float tiles_cost(bool f32, int64_t m, int64_t rows, float steps, int edge) {
  TileCost c = f32 ? (edge == kTile ? TileCost{4.f, 1.f, 1.f, 1.f}
                                    : edge == 128 ? TileCost{1.2f, 0.52f, 0.52f, 0.52f} : TileCost{1.f, 0.285f, 0.f, 0.f})
                   : (edge == kTile ? TileCost{11.6f, 1.f, 0.4f, 0.4f}
                                    : edge == 128 ? TileCost{3.9f, 0.81f, 0.31f, 0.57f} : TileCost{2.2f, 0.6f, 0.27f, 0.43f});
  // More output than the last-level cache holds: with rows of 4 KB or less the narrow tiles' ends cost more (d = 512 and
  // 1024, V = 80000 and 151936; most from four K-steps on), with longer ones the wide tiles' less (d = 2048 to 4096).
  if (!f32 && m * rows * 4 > ((int64_t)256 << 20)) {
    if (m <= 1024) c.ends += edge == kTile ? 0.4f : edge == 128 ? (steps >= 4.f ? 2.2f : 1.f) : 0.7f;
    else if (edge == kTile) c.ends -= 0.8f;
  }
  const int64_t m_tiles = (m + edge - 1) / edge, n_tiles = (rows + edge - 1) / edge;
  const int64_t slots = (int64_t)kComputeUnits * (kTile / edge);   // 256 / edge workgroups share a compute unit
  const int64_t rounds = m_tiles * n_tiles / slots;
  const float fill = (float)(m_tiles * n_tiles - rounds * slots) / (float)slots;   // of the last round
  const float round = c.ends + steps * c.step;
  if (rounds >= 4) return ((float)rounds + fill) * round;   // a partial round behind many overlaps them
  // the eight L2s hold 32 MB of operands; with 100 MB more next to nothing of a tile's is there
  const float beyond = ((float)(m + rows) * steps * 128.f / 1048576.f - 32.f) / 100.f;
  const float alone = c.near + (c.far - c.near) * (beyond < 0.f ? 0.f : beyond < 1.f ? beyond : 1.f);
  auto partial = [&](float n, float f) { return c.ends + n * (c.step * f > alone ? c.step * f : alone); };
  if (const int ks = edge == kTile ? dw_tail_slices(m_tiles, n_tiles, kComputeUnits) : 1; ks > 1) {
    const int64_t per_round = kComputeUnits / m_tiles;
    const float f = (float)(m_tiles * (n_tiles % per_round) * ks) / (float)kComputeUnits;
    // and the sum of the slices, with what their 64 MB push out of the caches for the kernels around it
    return (float)(n_tiles / per_round) * round + partial(steps / (float)ks, f) + (f32 ? 1.5f : 32.f) * f;
  }
  return (float)rounds * round + (fill > 0.f ? partial(steps, fill) : 0.f);
}
inline int cheapest_edge(bool f32, int64_t m, int64_t rows, float steps) {
  int best = kTile;
  float least = tiles_cost(f32, m, rows, steps, kTile);
  for (int edge : {128, 64}) {
    const float cost = tiles_cost(f32, m, rows, steps, edge);
    if (cost < least) {
      least = cost;
      best = edge;
    }
  }
  return best;
}
inline int dw_edge(bool f32, int64_t m, int64_t rows, int64_t n) {
  return cheapest_edge(f32, m, rows, (float)((n * (f32 ? 4 : 2) + 127) / 128));
}
// dH: m = d, n = token slots, contraction of `ksteps` 128-byte steps over the vocabulary that can be cut into
// slices (see DhSplit): the largest edge that fills the chip with slices of 32 K-steps and does not
// exceed the tokens by much, for fp32 as for bf16.  (An fp32 contraction that is too short to cut fills the rounds best
// with 64 wide tiles: n 6000 d 1024 V 500 58 us against 72 on edge 128.)  Edge 256 / 128 / 64, us (fp32 once took edge 64
// up to four rounds of 256 wide tiles):
//   bf16: n 1024 d 1024 V 20000 61.0 / 58.1 / 130    n 512 d 4096 V 32000 136 / 217 / 340    n 256 d 256 V 4096 24.5 / 15.0 / 12.4
//   fp32: n 4096 d 1024 V 32000 1839 / 1960 / 2150   n 1024 d 1024 V 16000 269 / 258 / 326   n 512 d 256 V 4096 56 / 29 / 20
//         n 4096 d 512 V 20000 607 / 620 / 671       n 512 d 512 V 20000 143 / 93 / 105      n 256 d 512 V 4096 60 / 31 / 22
inline int dh_edge(bool f32, int64_t m, int64_t n, int64_t ksteps) {
  const int64_t slices = ksteps / 32 > 0 ? ksteps / 32 : 1;
  if (f32 && slices == 1) return tiles_of(m, n, kTile) <= 4 * kComputeUnits ? 64 : kTile;
  if (n > 128 && tiles_of(m, n, kTile) * slices >= kComputeUnits) return kTile;
  if (n > 64 && tiles_of(m, n, 128) * slices >= kComputeUnits) return 128;
  return 64;
}

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

// ---- KV path ----

// Tile edge of the KV kernels: 64, 128 or 256, four wavefronts each.  The smaller the edge, the more operand bytes per
// flop (edge 256 is the only one that the vector L1 can feed at full matrix rate), but the more workgroups there are
// to fill the chip with, and the shorter a tile's serial K loop and epilogue are.  Spectral projection, d = 1024, us:
//     n            256   1024   2048   4096   8192  12000  16384  65536
//     edge 64     11.5   12.7   14.0   20.2   36.8   50.6   59.9    252
//     edge 128    14.3   15.3   15.7   17.2   25.3   35.9   44.5    179
//     edge 256    29.4   30.5   30.8   31.9   34.5   37.0   42.2    143
// (fp32, n = 1024: 26.8 / 66.8 / 239; n = 4096: 80 / 78 / 241.)  So: the smallest edge whose tiles run in one round, two to
// a compute unit.
// Beyond that the padding of the d columns counts: 320 columns are 512 in 256 wide tiles and 384 in 128 wide ones,
// 128 columns 256 and 128 (gate of 37065 x 320 94 -> 63 us, fp32 40000 x 320 354 -> 195, 262144 x 128 201 -> 147).
// In bf16 so do the rounds: 256 wide tiles have a compute unit each, and a round that is not full takes most of a full one's time;
// 128 wide ones take longer per round, the more so the longer the contraction, but half as long as that.  wide_cost and
// narrow_cost are fits, in full rounds of 256 wide tiles, to (training pair, us, edge 128 / 256):
//   d 1024: n 9000 262 / 288   12000 309 / 331   17000 414 / 501   20000 469 / 541   24000 555 / 587   28000 653 / 645   32768 774 / 726
//           36000 820 / 865   40000 912 / 911   49152 1099 / 1015   65536 1364 / 1317
//   d 2048: n 4500 394 / 387   8192 619 / 569   9000 708 / 774   10000 766 / 816   12000 891 / 872   16384 1168 / 1042   20000 1403 / 1349
//   d 512:  n 20000 206 / 236   32768 293 / 309   40000 349 / 421   65536 569 / 570   80000 695 / 721   120000 1015 / 1017
//   others: 12000 x 1536 603 / 685   30000 x 768 497 / 542   70000 x 256 281 / 359   200000 x 256 729 / 822
// and, the reconstruction counting half the K-steps as its tokens do (store and reconstruction): d 1024: n 32768 67 / 71   65536
// 123 / 126   100000 184 / 200   131072 274 / 253;   d 512: 100000 82 / 96   200000 158 / 177;   d 2048: 12000 80 / 86   24000 138 / 122.
// The choice is within 3 % of the better edge at all of these but one: the reconstruction of 100000 x 1024, a tie by the fits, is
// 9 % slower than it would be on edge 128.  (Lengths as a gate with a retain rate of 0.44 leaves them.  Longer ones favour edge 256:
// the reconstruction of 200000 x 512 alone, lengths in [0.8 d, d], 196 us on edge 128, 180 on 256.)
inline int kv_tile_edge(bool f32, int mode, int M, int64_t Nn, int K, int64_t cus) {
  auto tiles = [&](int edge) { return tiles_of(M, Nn, edge); };
  if (tiles(64) <= 2 * cus) return 64;
  if (tiles(128) <= (f32 && mode == 2 ? 8 : 2) * cus) return 128;
  int best = 256;
  auto padded = [&](int edge) { return (float)((M + edge - 1) / edge * edge) / tile_rate(edge, f32); };
  if (!f32) {
    auto rounds = [&](int edge, int64_t slots, float least) {   // a last round that is not full counts at least `least`
      const int64_t full = tiles(edge) / slots;
      const float rest = (float)(tiles(edge) % slots) / (float)slots;
      return (float)full + (rest > 0.f ? (rest > least ? rest : least) : 0.f);
    };
    const float steps = (float)(K / 64) * (mode == 2 ? 0.5f : 1.f);
    const float slope = 1.03f + 0.015f * steps, first = 0.45f - 0.0125f * steps;
    const float wide_cost = rounds(256, cus, 0.8f);
    const float narrow_cost = (slope < 1.3f ? slope : 1.3f) * rounds(128, 2 * cus, 0.5f) / 2 - (first > 0.f ? first : 0.f);
    best = narrow_cost < wide_cost ? 128 : 256;
  } else if (padded(128) < padded(256)) {
    best = 128;
  }
  return padded(64) < padded(best) ? 64 : best;
}

// Tiles that hold five K-steps in LDS instead of two and a half (bf16): where every tile has a compute unit for itself, so that
// nothing else covers an access to L2, which takes longer than the MFMAs of a K-step do, and the contraction has 16 K-steps or
// more.  Shorter ones end before the lead pays for the five requests in front of the first MFMA, and two or more tiles on a
// compute unit cover each other.  The ring / five stages, us:
//   gate   1024 x 1024 25.0 / 20.6   550 x 1024 24.5 / 19.9   1100 x 2048 51.0 / 45.4   4096 x 1024 36.2 / 34.5
//          (more tiles: 2048 x 1024 27.3 / 27.8, 4096 x 512 19.8 / 21.5; shorter: 2000 x 512 16.2 / 17.0)
//   store + reconstruction   1000 x 1024 26.1 / 23.4; on edge 128 no faster (3000 x 1024 28.3 / 28.2)
//   training pair   1024 x 1024 83.1 / 72.5   4096 x 1024 136.4 / 134.9
// Eight stages are no faster (gate 1024 x 1024 22.0).
constexpr int kStages = 5, kDeepSteps = 16;
inline bool kv_deep_tiles(int mode, int edge, int M, int64_t Nn, int K, int64_t cus) {
  return tiles_of(M, Nn, edge) <= cus && K / 64 >= kDeepSteps && (edge == 64 || (edge == 128 && mode != 2));
}

// The few-token kernel (16 tokens x 64 columns a workgroup) takes up to two workgroups per compute unit: every 16 tokens read all
// of the parameters again.  Gate of n tokens, copies and tiled products / these (us):
//   d 1024 bf16: n 16 27.4 / 15.7   n 256 28.3 / 17.1;   d 1024 fp32: n 16 54.3 / 23.6   n 512 58.3 / 39.4
// One per compute unit where the tiled products hold five K-steps (kv_deep_tiles), tiled / these:
//   d 1024: n 64 17.8 / 15.3   256 18.9 / 16.1   300 19.1 / 21.2   512 20.2 / 22.3;   d 2048: n 128 25.3 / 24.0   190 26.2 / 34.6
//   training pair: d 1024 n 256 70.1 / 65.9   400 65.4 / 77.7;   d 2048 n 256 93.3 / 124.5
constexpr int kFewCols = 64, kFewTok = 16;
inline bool kv_few_fits(bool f32, int64_t n, int d) {
  const int per_unit = !f32 && d / 64 >= kDeepSteps ? 1 : 2;
  return (n + kFewTok - 1) / kFewTok * (d / kFewCols) <= per_unit * (int64_t)kComputeUnits;
}

// Tile edge and slices of the parameter gradients' contraction over the tokens, in a launch of their own: as many slices as give one
// workgroup per compute unit, on the largest edge whose slices then keep 16 K-steps (of 128 bytes; edge 256: 32), else edge 64 with
// at least 2 each.
// dW alone / whole backward call, us, bf16 unless said, with the choice in brackets:
//     n x d           edge 256         edge 128          edge 64          (slices giving 256 workgroups, or the best)
//     32768 x 1024    [72.6 / 611]     99.6 / 638        208 / 867
//     8192 x 2048     [63.4 / 528]     79.2 / 555        113 / 626
//     4096 x 1024     23.4 / 177       [18.3 / 156]      30.6 / 181
//     512 x 1024      17.4 / 117       11.3 / 100        [9.8 / 93]
//     8192 x 256      18.0 / 115       11.5 / 102        [9.6 / 92]
//     300 x 128 fp32  20.6 / 83        9.9 / 63          [7.6 / 59]
// Training pair, edge 256 / 128, where slices of 256 wide tiles have 16 K-steps: 4096 x 2048 346.5 / 309.7, 16384 x 1024
// 398.5 / 383.0, fp32 8192 x 1024 978 / 943; 23: 6000 x 2048 474 / 449, 24000 x 1024 596 / 583; 32: 8192 x 2048 568 / 570,
// 32768 x 1024 708 / 707, fp32 16384 x 1024 1874 / 1853; 64: 65536 x 1024 1317 / 1364.
struct KvTail {
  int edge = 0, slices = 0;
};
inline KvTail kv_gradient_slices(bool f32, int64_t n, int d) {
  const int64_t ksteps = (n + kTile - 1) / kTile * kTile * (f32 ? 4 : 2) / 128;
  KvTail t;
  for (int edge : {256, 128, 64}) {
    const int64_t side = (d + edge - 1) / edge;
    int64_t ks = (256 + side * side - 1) / (side * side);
    const bool last = edge == 64;
    if (last && ks > ksteps / 2) ks = ksteps / 2;
    if (ks < 1) ks = 1;
    t.edge = edge;
    t.slices = (int)ks;
    if (last || ksteps / ks >= (edge == 256 ? 32 : 16)) break;
  }
  return t;
}

// What follows g_x~ in a backward call (dx, both parameter gradients, the sums of their slices, db) as one launch: none of them waits
// for another, each leaves compute units idle by itself, and a launch costs its 4 us wherever it is put.  All on tiles of one edge.  The
// last workgroup of a gradient tile reads all its slices alone, so there are to be few of them, and of equal length with the rest.
// Training pair, us, launches of their own / one (bf16; edge, slices: of launches of their own / of one):
//     n x d        us             edge, slices           n x d        us             edge, slices
//     64 x 64      45.6 / 39.3    64, 2 / 64, 1          1024 x 1024  76.1 / 68.4    64, 1 / 64, 1
//     700 x 256    49.3 / 42.5    64, 6 / 64, 1          4096 x 1024  145 / 134      128, 4 / 128, 2
//     2000 x 512   65.8 / 59.6    64, 4 / 64, 2          1500 x 1536  153 / 130      64, 1 / 128, 1
//     5000 x 256   62.6 / 58.3    64, 16 / 64, 5         8192 x 1024  218 / 203      128, 4 / 128, 2
//     32768 x 256  141 / 136      64, 16 / 64, 16        2048 x 2048  201 / 199      128, 1 / 128, 1
//     16384 x 384  125 / 120      64, 8 / 64, 8          14000 x 640  213 / 195      128, 11 / 128, 6
// Other choices: 4096 x 1024 with 1, 3, 4, 8 slices 140, 137, 145, 180; 1024 x 1024 on edge 128 79, 2048 x 1024 107 instead of 100;
// 1500 x 1536 on edge 64 140.  Beyond the work and the slices that it stops at: 3000 x 2048 (71) 256 / 259, 16384 x 1024 397 / 391,
// 65536 x 64 (64 slices) 122 / 124, 16700 x 64 63 / 64; on edge 128 with 9 to 16 slices 16384 x 448 141 / 144, 32768 x 448 261 / 283,
// 32768 x 384 224 / 234, 40000 x 320 240 / 244.
// fp32 keeps the slices that its sums had (longer ones raise the error of dU from 2.28e-6 to 2.49e-6 at 4096 x 1024), and so edge
// 64 (2048 x 1024 with 4 slices on edge 128: 305 / 370; 2000 x 256, 16 slices, 66.5 / 72.9).  Launches of their own / one:
//     100 x 64   41 / 36    40 x 192  40.7 / 38.6    300 x 128 40.7 / 38.2    2000 x 576  163 / 147    1000 x 768  139 / 122
//     1500 x 448 97 / 85    300 x 1024 123 / 119     600 x 1280 202 / 185     1000 x 1152 272 / 248
// Of few tokens, whose dx stays apart, only the gradients are left, and their slices go through memory instead of staying in L2:
//     300 x 256 45.0 / 46.9    512 x 320 54.4 / 55.9    16 x 512 52.6 / 57.3    16 x 640 62.1 / 67.1    100 x 448 53.9 / 54.6
// edge 0: launches of their own.
inline KvTail kv_tail(bool f32, int64_t n, int d, const KvTail& own) {
  const int kMostWork = 48;
  if (own.edge > (f32 ? 64 : 128)) return {};
  if (f32 && own.slices > 1 && own.slices * d > 1024 && kv_few_fits(f32, n, d)) return {};
  const int esz = f32 ? 4 : 2;
  const int64_t ksteps = (n * esz + 127) / 128, dx_steps = ((int64_t)d * esz + 127) / 128;
  // K-steps of a place for a workgroup (256 / edge of them on a compute unit), were all equally loaded
  auto work = [&](int edge) {
    return (2 * tiles_of(d, d, edge) * ksteps + tiles_of(d, n, edge) * dx_steps) / (kComputeUnits * (256 / edge));
  };
  KvTail t;
  t.edge = !f32 && work(128) >= 16 ? 128 : 64;
  const int64_t w = work(t.edge), steps = w > 12 ? w * 4 / 3 : 16;   // of a slice
  t.slices = own.slices;   // never more: the scratch memory is sized for these, and grows with n
  if (!f32 && (ksteps + steps - 1) / steps < own.slices) t.slices = (int)((ksteps + steps - 1) / steps);
  return w <= kMostWork && t.slices <= (f32 || t.edge == 128 ? 8 : 16) ? t : KvTail{};
}
// Whether dx stays a launch of its own before it (pair, us, launches of their own / dx within / apart):
//  - few tokens, bf16 from 2048 components on: sixteen wavefronts share the contraction of the product of few tokens, one has it in
//    a tile.  16 tokens, d 1024 / 2048 / 4096, apart / within: 52.6 / 49.2, 85.2 / 84.3, 188 / 190; 1 x 8192: 442 / 491.  In fp32 it also
//    keeps the sums short (300 x 128: error 3.98e-7, within 4.58e-7).
//  - bf16 tiles that hold five K-steps by themselves (kv_deep_tiles), whose contraction is longer than all the rest:
//    100 x 3072 145 / 148 / 144   256 x 4096 208 / 212 / 200   100 x 5120 259 / 292 / 260   100 x 8192 499 / 544 / 490;
//    not 256 x 2560 140 / 137
//  - fp32 tiles that would start in a last round of places that they have to themselves: they share compute units there, four to one,
//    and others idle.  800 x 960 162 / 173 / 160   600 x 1408 216 / 229 / 214   400 x 1536 216 / 226 / 212   256 x 2560 356 / 377 / 354;
//    with a fuller round 400 x 1792 256 / 240, with more tiles of dx than compute units 1200 x 896 223 / 205, 800 x 1280 291 / 271
inline bool kv_tail_dx_apart(bool f32, int64_t n, int d, const KvTail& t) {
  if (kv_few_fits(f32, n, d)) return f32 || d > 2048;
  if (!f32) return d >= 3072 && kv_deep_tiles(3, kv_tile_edge(false, 3, d, n, d, kComputeUnits), d, n, d, kComputeUnits);
  const int64_t places = kComputeUnits * (256 / t.edge), dx = tiles_of(d, n, t.edge), all = dx + 2 * t.slices * tiles_of(d, d, t.edge);
  return dx <= kComputeUnits && all > places && all % places < places / 2;
}
inline int64_t kv_tail_counters(int64_t d) { return 2 * ((d + 63) / 64) * ((d + 63) / 64); }

// Whether the few-token product of the logits makes their mask too (kv_few_mask_kernel), instead of a launch for it.  That launch costs its
// 2.5 us where calls are short enough to wait for each other's launches (20 us of gate and store, less of a gate alone), and next to
// nothing in a captured graph.  The workgroup that is last has 16 tokens to itself, behind stores that have gone through to memory: 0.2 us
// for a few short rows, 3 us for many long ones, more with soft outputs to write.  So: where a gate alone is not slower, by tokens x
// components for each group of 256 components.  Gate alone / with the store, us, launch : same launch, bf16:
//   16 x 256   14.6 : 11.9  22.6 : 20.2      256 x 512   - : -        22.8 : 20.2     540 x 448  14.3 : 12.7
//   64 x 640   13.1 : 12.6  20.9 : 18.2      64 x 768    13.3 : 13.3  20.8 : 18.2     16 x 896   14.4 : 14.4  22.7 : 20.1
//   32 x 1024  15.2 : 15.1  22.1 : 20.0      not  1000 x 448 14.8 : 16.1   240 x 704 14.3 : 15.2   160 x 768 13.3 : 14.2  20.2 : 18.6
//   64 x 896 14.9 : 15.4  20.2 : 18.8   128 x 1024 15.5 : 16.7  20.5 : 20.9
// fp32:  300 x 256 14.6 : 12.5  23.1 : 20.3   64 x 448 15.0 : 15.0  22.8 : 20.3   not 300 x 448 15.5 : 15.9   16 x 640 17.4 : 17.8  20.9 : 21.4
//   300 x 768 20.4 : 21.7
// with soft outputs (training pair):  300 x 128 fp32 47.3 : 45.0  4096 x 64 43.1 : 40.3  1000 x 256 51.0 : 48.4  600 x 256 fp32 49.2 : 49.8
//   256 x 512 49.5 : 49.9  128 x 1024 55.6 : 57.7  700 x 512 58.4 : 61.0
constexpr int kKvFewMask = 1024;
inline bool kv_mask_with_logits(int esz, int64_t n, int d, bool soft) {
  constexpr int64_t kMost[2][kKvFewMask / 256] = {{512 << 10, 256 << 10, 64 << 10, 32 << 10}, {512 << 10, 48 << 10, 0, 0}};
  return soft ? d * esz <= 512 : d <= kKvFewMask && n * d <= kMost[esz == 4][(d - 1) / 256];
}

}  // namespace lmhead
