// Internal declarations of the KV-compression path: workspace layout and launcher prototypes.
#pragma once

#include "../../include/dynakv.h"
#include "common.h"

namespace lmhead {

constexpr int kKvMaxD = 8192;
constexpr int kKvRetainBlocks = 2048;   // blocks of the retain-rate sums: 256 threads each, one resident round
constexpr int kKvScanBlock = 256;    // tokens per block of the offset scan
constexpr int kKvCountBlocks = 256;    // most blocks of the counts per contraction length

// Sticky error bits of this path (same header word as the LM-head path).
constexpr int kErrKvCount = 4;       // a k outside [0, d]
constexpr int kErrKvCapacity = 8;    // a segment beyond the capacity of the store

struct KvLayout {
  int esz;
  int64_t n, d;
  int64_t ncap;      // n rounded up to the tile
  int64_t dp;        // d rounded up to the tile
  int nbuckets;      // K-steps a token can need, plus one: d * esz / 128 + 1
  size_t hdr, Ufrag, Wfrag, logits, order, pos_off, pos_len, hist, blocksum, red, total;
};

static inline KvLayout make_kv_layout(const dynakv_desc* d) {
  KvLayout L{};
  L.esz = d->dtype == LMHEAD_BF16 ? 2 : 4;
  L.n = d->n;
  L.d = d->d;
  L.ncap = (int64_t)round_up((size_t)L.n, kTile);
  L.dp = (int64_t)round_up((size_t)L.d, kTile);
  L.nbuckets = (int)(L.d * L.esz / 128) + 1;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += round_up(bytes, 256);
    return o;
  };
  L.hdr = take(sizeof(WsHeader));
  L.Ufrag = take((size_t)L.d * L.d * L.esz);   // for the one-kernel gate
  L.Wfrag = take((size_t)L.d * L.d * L.esz);
  L.logits = take((size_t)L.ncap * L.d * 4);
  L.order = take((size_t)L.ncap * 4);
  L.pos_off = take((size_t)L.ncap * 4);
  L.pos_len = take((size_t)L.ncap * 4);
  L.hist = take((size_t)kKvCountBlocks * L.nbuckets * 4);   // tokens per block and bucket
  L.blocksum = take((size_t)(L.ncap / kKvScanBlock + 2) * 8);
  L.red = take((size_t)kKvRetainBlocks * 2 * 8);      // per-block partial sums of the retain rate
  L.total = off;
  return L;
}

// Workspace of the gate's backward pass (dynakv_gate_bwd).  The two token-major gradients g_l and
// g_xt are kept in the storage type.
struct KvBwdLayout {
  int esz;
  int64_t n, d, ncap, dp;
  int edge, ksplit;  // tile edge of dW / dU and slices of their contraction over the tokens
  bool tail;         // they, dx and db in one launch
  int nblk;          // workgroups of the mask backward kernel = rows of the db partial sums
  size_t hdr, logits, gl, gxt, part, dbpart, done, total;
};

// Workgroups of the mask backward kernel: four 256-thread workgroups fit a compute unit (128 VGPRs),
// so 1024 is one resident round on 256 compute units; each wavefront loops over its share of tokens.
constexpr int kKvBwdMaxBlocks = 1024;

static inline KvBwdLayout make_kv_bwd_layout(const dynakv_desc* d) {
  KvBwdLayout L{};
  L.esz = d->dtype == LMHEAD_BF16 ? 2 : 4;
  L.n = d->n;
  L.d = d->d;
  L.ncap = (int64_t)round_up((size_t)L.n, kTile);
  L.dp = (int64_t)round_up((size_t)L.d, kTile);
  const KvTail own = kv_gradient_slices(L.esz == 4, L.n, L.d);
  L.edge = own.edge;
  L.ksplit = own.slices;
  const int part_slices = L.ksplit;
  if (const KvTail t = kv_tail(L.esz == 4, L.n, L.d, own); t.edge) {
    L.tail = true;
    L.edge = t.edge;
    L.ksplit = t.slices;
  }
  {
    const int64_t blocks = (L.n + 3) / 4;
    L.nblk = (int)(blocks < kKvBwdMaxBlocks ? blocks : kKvBwdMaxBlocks);
  }
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += round_up(bytes, 256);
    return o;
  };
  L.hdr = take(sizeof(WsHeader));
  L.logits = take((size_t)L.ncap * L.d * 4);
  L.gl = take((size_t)L.ncap * L.d * L.esz);
  L.gxt = take((size_t)L.ncap * L.d * L.esz);
  L.part = take((size_t)2 * part_slices * L.d * L.d * 4);   // the slices of both gradients
  L.dbpart = take((size_t)L.nblk * L.d * 4);
  L.done = take((size_t)kv_tail_counters(L.d) * 4);
  L.total = off;
  return L;
}

// Plain contraction on the MFMA tile core with a transposed store:
//   out[row(n)][m] = sum_k A[m][k] * Bop[n][k],  m < M, n < Nn.
// mode 0/1: Bop rows are dense rows of B (pitch ldB), row(n) = n.  The output is the storage type
//           (out_e) or fp32 (out_f), whichever is non-null.
// mode 3:   as mode 0 for the transposed parameter matrix.
// A is the parameter matrix as the caller has it: [K x M], mode 3: [M x K].
// mode 2:   ragged rows: Bop[n] = the pos_len[n] bytes of the packed store at byte offset pos_off[n],
//           zero beyond; row(n) = order[n] (< 0: no token); the tile's step count follows its
//           first row, the longest (the three arrays are written by launch_kv_order or launch_kv_group).
struct KvGemmArgs {
  int mode;
  const void* A;        // pitch ldA
  int64_t bytesA;       // readable at A; what lies beyond counts as zeros
  int64_t ldA;
  const void* B;        // dense rows (mode 0/1) or the packed store (mode 2)
  int64_t ldB;
  int64_t bytesB;       // mode 2: bytes readable at B
  int M;                // output columns (d)
  int64_t Nn;           // tokens
  int K;                // contraction length in elements (d)
  const int32_t* order;     // mode 2
  const uint32_t* pos_off;  // mode 2
  const int32_t* pos_len;   // mode 2
  const int32_t* outside;   // mode 2, unless null: launch_kv_group's flags, from which the header is set
  int groups;
  void* out_e;
  float* out_f;
  int64_t ldo;
  bool clear;           // the header is cleared
  bool accumulate;      // dense modes: the tile is added to what the output holds (rounded once more for bf16)
  WsHeader* hdr;
  int walk_len;         // set by the launcher: length of the tile walk (tile_map.h)
};
hipError_t launch_kv_gemm(int dtype, const KvGemmArgs& a, hipStream_t s);

// out = the n rows of row_bytes (a multiple of 16), `pitch` bytes apart, one behind the other.
hipError_t launch_kv_dense(const void* x, int64_t pitch, int64_t n, int row_bytes, void* out, hipStream_t s);

// out[n][j] = sum_k x[n][k] M[k][j], or with kFewRows sum_k x[n][k] M[j][k], for few tokens: M [d x d] as the caller has
// it (no copy), 16 tokens x 64 columns per workgroup.  out: dense rows of d, in the storage type or (kFewWide) fp32; kFewAdd: added to,
// storage type only.  Clears the header unless null.
constexpr int kFewRows = 1, kFewAdd = 2, kFewWide = 4;
struct KvFewArgs {
  const void* x;
  int64_t ldx;
  const void* M;
  int n, d;
  void* out;
  WsHeader* hdr;
  int32_t* clear;      // unless null: one counter per 16 tokens, set to 0
  int flags;
};
// The arguments of a launch come from host memory, a line at a time, and each of these products waits for them: with the next line in it
// a gate of 32 x 1024 in fp32 took 23.4 us instead of 22.9.
static_assert(sizeof(KvFewArgs) <= 64, "one line");
// The product is the gate's logits (kFewWide), and the last workgroup of 16 tokens makes their mask (launch_kv_mask, d up to kKvFewMask).
struct KvFewMask {
  int32_t* k;
  int32_t* done;       // the counters, cleared by a launch before
  const float* bias;
  const void* xt;
  float* m;
  void* xhat;
  float tau;
  bool literal;
};
hipError_t launch_kv_few(int dtype, const KvFewArgs& a, hipStream_t s, const KvFewMask* mask = nullptr);

// The whole gate of many tokens in one kernel (dynakv_gate.hip), for callers that want x~ and k only.  Ufrag, Wfrag: the
// parameter matrices in fragment order (KvCopy, W's flipped when `literal`).
struct KvGateArgs {
  const void* x;
  int64_t ldx;
  const void* Ufrag;
  const void* Wfrag;
  const float* bias;
  int64_t n;
  float tau;
  int literal;
  void* xt;
  int32_t* k;
};
// From this many tokens on.  Its workgroups take 64 tokens (128 at d = 512) through everything, 60 us a round, so with less than
// half a round the separate kernels with their smaller tiles win.  Whole call, us, separate kernels / this one:
//   d 1024: n 8192 53.8 / 60.2   9000 69.4 / 60.9   10240 72.1 / 61.9   12000 76.7 / 64.7   16384 89.3 / 71.9   20000 115 / 121
//           32768 176 / 136   65536 342 / 258   262144 1309 / 1002
//   d 512:  n 8192 29.4 / 32.7   10000 33.9 / 33.6   12000 35.5 / 35.4   16384 42.0 / 37.4   32768 68.8 / 45.2   65536 132 / 83
//           262144 539 / 312
// (20000 x 1024 begins a second round of 57 workgroups.)
// bf16 at 512 and 1024 only: the tile is laid out for a whole token row in LDS next to 128 accumulators a lane, 64 tokens of
// 1024 or 128 of 512 components.  A row of 2048 leaves room for 32 tokens, i.e. twice the parameter stream per token, which
// is the bound; 256 and 768 would take other piece and lane maps, unwritten since no workload has such a d at
// these lengths, and fp32 is bound by the matrix rate, which the separate kernels come close to (135 of 157 TFLOP/s).
constexpr int kKvGateFrom = 10240;
constexpr int kKvGateWaves = 8;
bool kv_gate_fits(int dtype, int64_t n, int d, int64_t ldx);
hipError_t launch_kv_gate(const KvGateArgs& a, int d, hipStream_t s);

// Softmax over the gate logits (+ bias), the cumulative mask, the threshold count and the
// optional training outputs.
hipError_t launch_kv_mask(int dtype, const float* logits, const float* b, const void* xt, int64_t n, int d,
                          float tau, bool literal, int32_t* k, float* m, void* xhat, hipStream_t s);

// off = off_base + exclusive prefix sum of roundup(k, 8), and the segments are copied; clears the header.
hipError_t launch_kv_store(int dtype, const void* xt, const int32_t* k, int64_t n, int d, int64_t off_base,
                           int64_t* off, void* packed, int64_t capacity, int64_t* blocksum, WsHeader* hdr,
                           hipStream_t s);

// Tokens per K-step bucket (ceil(k * esz / 128)), counted in `blocks` blocks of per_block tokens:
// hist[block][bucket].  Blocks of 1024 tokens, larger ones beyond kKvCountBlocks of them.
struct KvCount {
  const int32_t* k;
  int64_t n;
  int d, nbuckets, blocks, per_block;
  int32_t* hist;
};
static inline KvCount make_kv_count(const int32_t* k, int64_t n, int d, int nbuckets, int32_t* hist) {
  const int64_t per = (n + (int64_t)kKvCountBlocks * 1024 - 1) / ((int64_t)kKvCountBlocks * 1024) * 1024;
  return {k, n, d, nbuckets, (int)((n + per - 1) / per), (int)per, hist};
}

// A parameter matrix (bf16, d x d, d a multiple of 128) as the MFMA fragments in the order in which kv_gate_kernel's
// wavefronts consume them, ((w * d/32 + s) * d/128 + i) KB + 16 lane bytes holding in[k][c] for the 8 values
// k = 32 s + 8 (lane / 16) + [0, 8) and column c = position d/8 w + d/32 ((lane % 16) / 4) + 4 i + lane % 4
// (flipped: c = d - 1 - position).
struct KvCopy {
  const void* in;
  int d;
  void* out;
  bool flipped;
};
struct KvPrepareArgs {
  WsHeader* hdr;       // cleared unless null
  KvCopy job[2];
  int njobs;
  KvCount count;       // blocks = 0: nothing to count
};
hipError_t launch_kv_prepare(int esz, const KvPrepareArgs& a, hipStream_t s);

// order = tokens sorted by descending number of K-steps, padded with -1 up to ncap; pos_off / pos_len = byte offset and
// byte length (k rounded up to the granule) of each sorted position's segment in a store of `bytes` readable bytes
// (0x80000000 / 0 for padding; 0x80000000 for segments that do not lie inside it, which also set the error word).
// The counts have been made by launch_kv_prepare.
hipError_t launch_kv_order(int dtype, const KvCount& c, const int64_t* off, int64_t bytes, int64_t ncap, int32_t* order,
                           uint32_t* pos_off, int32_t* pos_len, WsHeader* hdr, hipStream_t s);

// The same in one launch: the tokens are sorted within groups of kKvGroup, whose tiles of `edge` tokens are dealt out in turn.
// outside[group]: whether a segment of the group does not lie inside the store.
constexpr int kKvGroup = 2048;
constexpr int64_t kKvGroupTo = 32768;
// fp32 products of 200 us and more stay with the sort of all the tokens: there the evener tiles are worth more than the launch.
// Reconstruction, lengths uniform in [0, d], us, all / groups:  fp32 3000 x 4096 503 / 552   24000 x 2048 957 / 1025   9000 x 2048
// 397 / 418   24000 x 1024 229 / 236   16384 x 1024 173 / 169   4500 x 512 45 / 41;   bf16 24000 x 2048 118 / 120   32768 x 4096
// 555 / 524   16384 x 1024 38 / 34   3000 x 512 13.6 / 10.7.
inline bool kv_group_fits(int esz, int64_t n, int64_t d) { return n <= kKvGroupTo && (esz == 2 || n * d * d <= (int64_t)1 << 34); }
static_assert(kKvGroup % kTile == 0 && kKvGroupTo / kKvGroup <= kKvCountBlocks, "whole tiles; the flags take the counts' place");
hipError_t launch_kv_group(int dtype, const int32_t* k, const int64_t* off, int64_t n, int d, int64_t bytes, int nbuckets, int edge,
                           int32_t* order, uint32_t* pos_off, int32_t* pos_len, int32_t* outside, hipStream_t s);

// Retain rates; clears the header.
hipError_t launch_kv_retain(const int32_t* k, const float* m, int64_t n, int d, float alpha, float* out,
                            float* g_m, double* red, WsHeader* hdr, hipStream_t s);

// Backward of softmax + cumulative mask + soft gating for every token (one wavefront per token):
//   q = g_xhat * xt + g_m + g_m_const;  r = inclusive prefix sums of q;  g_l = p * (r - sum p r);
//   a = g_xhat * m.
// g_l goes to gl (gate column order) and a to a_out, both [n x d] in the storage type; dbpart
// receives one row of column sums of g_l per workgroup (nblk rows, launch grid = nblk).  clear[0 .. nclear) is set to 0.
hipError_t launch_kv_mask_bwd(int dtype, const float* logits, const float* b, const void* xt, const void* g_xhat,
                              const float* g_m, float g_m_const, int64_t n, int d, bool literal, void* gl,
                              void* a_out, float* dbpart, int nblk, int32_t* clear, int nclear, hipStream_t s);

// db (+)= the column sums of dbpart [db_rows x d]; with slices > 1 also dW (+)= the sum of the first `slices` d x d matrices of
// part and dU (+)= that of the next ones.  Fixed order.
struct KvSums {
  const float* dbpart;
  int db_rows;
  const float* part;
  int slices, d;
  float *db, *dW, *dU;
  bool accumulate;
};
// The sum of a column's rows, by kSumWaves chains of every kSumWaves-th row, kSumBatch loads at a time.  The caller makes Q of the
// chains, first and every kSumWaves / Q after it, and stores them `to_step` floats apart.
constexpr int kSumWaves = 16, kSumBatch = 8;
template <int Q>
__device__ inline void column_sums(const float* __restrict__ p, int64_t pitch, int64_t rows, int first, float* to, int to_step) {
  constexpr int kStep = kSumWaves / Q;
  float t[Q][kSumBatch] = {};
  int64_t r0 = first;
  if constexpr (Q > 1)
    for (; r0 + (Q - 1) * kStep + (kSumBatch - 1) * kSumWaves < rows; r0 += kSumWaves * kSumBatch) {
      float v[Q][kSumBatch];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int u = 0; u < kSumBatch; ++u) v[q][u] = p[(r0 + q * kStep + u * kSumWaves) * pitch];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int u = 0; u < kSumBatch; ++u) t[q][u] += v[q][u];
    }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    int64_t r = r0 + q * kStep;
    for (; r + (kSumBatch - 1) * kSumWaves < rows; r += kSumWaves * kSumBatch) {
      float v[kSumBatch];
#pragma unroll
      for (int u = 0; u < kSumBatch; ++u) v[u] = p[(r + u * kSumWaves) * pitch];
#pragma unroll
      for (int u = 0; u < kSumBatch; ++u) t[q][u] += v[u];
    }
    for (; r < rows; r += kSumWaves) t[q][0] += p[r * pitch];
#pragma unroll
    for (int o = kSumBatch / 2; o > 0; o >>= 1)
#pragma unroll
      for (int u = 0; u < o; ++u) t[q][u] += t[q][u + o];
    to[q * to_step] = t[q][0];
  }
}

hipError_t launch_kv_sums(const KvSums& a, hipStream_t s);

// What follows g_x~ in a backward call, in one launch (kv_tail): the dense product `dx` (mode 3; Nn 0: without it), both gradients with
// the sum of their slices (role 2; g.done: their counters, cleared), and the column sums of q (its slices are not looked at).
hipError_t launch_kv_tail(int dtype, const KvGemmArgs& dx, const GemmTArgs& g, const KvSums& q, hipStream_t s);

}  // namespace lmhead
