// Matrix-core kernels of the KV-compression path, built on GemmTile (gemm_core.h):
//   mode 0  spectral projection     x~ = x U                      (Eq. 1)
//   mode 1  gate logits             x~ W          (fp32, bias added by the mask kernel; Eq. 5)
//   mode 2  dynamic low-rank reconstruction  x_bar = x^[0:k] U^-1[0:k, :]   (Eq. 3)
//   mode 3  the two token-major products of the gate's backward pass (M^T in place of M), optionally added to what
//           the output holds
// All are  out[row(n)][m] = sum_k A[m][k] Bop[n][k]  with the parameter matrix on the MFMA M axis and tokens on N, as in the
// LM-head kernels.  It is taken as the caller has it, K-major in modes 0 to 2: the launch that made transposed copies was
// 4.5 us (bf16 gate of 4096 x 1024 42.2 -> 37.6 us, with the gradients' copies the training pair 166 -> 148).  The
// parameter matrix (2 MB at d = 1024) stays in every XCD's L2; the token rows stream through once
// per XCD because an XCD runs all M tiles of a token tile together (tile_map.h).
//
// Mode 2 reads token rows of differing length straight from the packed store: row n of a tile is
// the segment of token order[n] (its byte offset and length come with it in pos_off / pos_len),
// loads beyond the segment's end fetch zeros (GemmTile's kMaskB), and the tile runs as many
// K-steps as its first token needs: `order` lists tokens by descending step count, so that is
// the tile's maximum and tiles of short tokens are short.
#include "dynakv_mask.h"
#include "gemm_t.h"

#include <type_traits>

namespace lmhead {

namespace {

constexpr int kKvMapBx = 4, kKvMapBy = 4;

// Workgroups of one tile edge that share a compute unit (bound by LDS: five slots of edge x 128 bytes each, or both operands' stages).
constexpr int wg_per_cu(int edge, int stages) { return stages ? 640 / (edge * stages) : 256 / edge; }

typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;

template <typename E, int Edge, int Mode, int Stages>
using KvTile = GemmTile<E, Edge, Edge, 2, 2, /*kLeadB=*/true, /*kMaskB=*/Mode == 2,
                        /*kTransA=*/Mode != 3, /*kTransB=*/false, /*kWalk=*/false, Stages>;

// One output tile; `wg` is the tile's position in the XCD-aware walk.
template <typename E, int Edge, int Mode, int Stages>
__device__ inline void kv_tile(const KvGemmArgs& a, int wg, char* smem) {
  using G = KvTile<E, Edge, Mode, Stages>;
  constexpr bool kTA = Mode != 3;
  constexpr int ESZ = Elem<E>::size;
  const int mtiles = (a.M + G::BM - 1) / G::BM;
  const int ntiles = (int)((a.Nn + G::BN - 1) / G::BN);
  int mt, nt;
  if (!xcd_tile_coords(wg, mtiles, ntiles, kKvMapBx, kKvMapBy, mt, nt)) return;
  if constexpr (Mode == 2) {
    // Token tiles come in order of falling step count: they are dealt out to the XCDs in turn.  (In contiguous ranges
    // the first XCD had the longest eighth of the tokens: 262144 tokens, retain rate 0.44: 491 us, now 392.)
    const int per = ntiles / kNumXcd;
    if (nt < per * kNumXcd) nt = nt % per * kNumXcd + nt / per;
  }
  const int64_t n0 = (int64_t)nt * G::BN;
  const int m0 = mt * G::BM;
  const int64_t pitchA = a.ldA * ESZ;

  uint32_t offA[G::A_LD], offB[G::B_LD];
  int limB[G::B_LD];
#pragma unroll
  for (int q = 0; q < G::A_LD; ++q) {
    const int row = kTA ? G::ldT_row(q) : G::ldA_row(q);
    offA[q] = (uint32_t)(row * pitchA) + (kTA ? G::ldT_byte(row) : G::ld_byte(row));
  }
  const char* Bbase;
  uint32_t bytesB;
  int ksteps;
  if constexpr (Mode == 2) {
#pragma unroll
    for (int q = 0; q < G::B_LD; ++q) {
      const int row = G::ldB_row(q);
      offB[q] = a.pos_off[n0 + row] + G::ld_byte(row);       // stays outside the buffer for padding rows
      limB[q] = a.pos_len[n0 + row] - G::ld_byte(row);
    }
    ksteps = (a.pos_len[n0] + G::KB - 1) / G::KB;
    Bbase = static_cast<const char*>(a.B);
    bytesB = (uint32_t)a.bytesB;
  } else {
    const int64_t pitchB = a.ldB * ESZ;
    const int last = (int)min((int64_t)G::BN - 1, a.Nn - 1 - n0);   // rows past the end re-read the last one
#pragma unroll
    for (int q = 0; q < G::B_LD; ++q) {
      const int row = G::ldB_row(q);
      offB[q] = (uint32_t)(min(row, last) * pitchB) + G::ld_byte(row);
      limB[q] = 0;
    }
    ksteps = a.K * ESZ / G::KB;
    Bbase = static_cast<const char*>(a.B) + n0 * pitchB;
    bytesB = 0x7fffffffu;
  }

  // output row of tile column threadIdx.x (fetched now, used after the main loop)
  int my_row = -1;
  if (threadIdx.x < G::BN) {
    if constexpr (Mode == 2)
      my_row = a.order[n0 + threadIdx.x];
    else
      my_row = n0 + threadIdx.x < a.Nn ? (int)(n0 + threadIdx.x) : -1;
  }

  typename G::Acc acc;
  G::zero(acc);
  const int64_t atA = (int64_t)m0 * (kTA ? ESZ : pitchA);
  G::run_ragged(acc, static_cast<const char*>(a.A) + atA, offA, (uint32_t)(a.bytesA - atA),
                kTA ? (uint32_t)(G::KROWS * pitchA) : (uint32_t)G::KB, Bbase, offB, limB, bytesB, ksteps, smem);

  // The tile leaves through LDS as [n][m] rows of fp32 (as many tile columns per phase as fit) so that
  // each output row segment is written with 16 bytes per lane for fp32 and 8 for bf16, a whole
  // number of rows per wavefront instruction.
  constexpr int JG = G::LDS_BYTES >= G::BN * (G::BM * 4 + 16) + G::BN * 4 ? G::TN : G::TN / 2;   // blocks per wave and phase
  constexpr int NPH = G::TN / JG;                 // phases
  constexpr int NCOL = G::WGN * JG * G::NB;       // tile columns staged per phase
  constexpr int P = G::BM * 4 + 16;               // staging row pitch in bytes
  constexpr int CH = G::BM * 4 / 16;              // lanes per staged row
  constexpr int RPI = 64 / CH;                    // staged rows per wavefront instruction
  constexpr int RPW = NCOL / G::NWAVES;           // staged rows per wave and phase
  static_assert(NCOL * P + G::BN * 4 <= G::LDS_BYTES && G::TN % JG == 0, "staging fits in LDS");
  static_assert(64 % CH == 0 && RPW % RPI == 0 && RPW * NPH <= 64, "row mapping");
  int* rows_lds = reinterpret_cast<int*>(smem + NCOL * P);
  if (threadIdx.x < G::BN) rows_lds[threadIdx.x] = my_row;
  // staged row -> tile column
  auto tile_col = [&](int phase, int r) {
    return (r / (JG * G::NB)) * G::WN + phase * (JG * G::NB) + r % (JG * G::NB);
  };
  const int h = G::lane() / CH;                   // which of the instruction's rows this lane works on
  const int c = G::lane() % CH;                   // its 16-byte chunk of the row = 4 output columns
  const int m = m0 + c * 4;
  constexpr int IPW = RPW / RPI;                  // instructions per wave and phase
  using OldT = typename std::conditional<ESZ == 2, bf16x4_t, f32x4_t>::type;
  const bool accumulate = Mode != 2 && a.accumulate && m < a.M;
#pragma unroll
  for (int jg = 0; jg < NPH; ++jg) {
    // When the tile is added to what the output holds, the old values of all the rows this wave writes
    // in this phase are requested now, so that their latency runs under the staging of the tile and is
    // paid once per phase.  (Dense modes only: the output row of a staged row is n0 + its tile column.)
    OldT oldv[IPW];
    if constexpr (Mode != 2) {
      if (accumulate) {
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
          const int64_t row = n0 + tile_col(jg, (G::wave() + G::NWAVES * i) * RPI + h);
          oldv[i] = OldT{};
          if (row < a.Nn) oldv[i] = *reinterpret_cast<const OldT*>(static_cast<const char*>(a.out_e) + (row * a.ldo + m) * ESZ);
        }
      }
    }
#pragma unroll
    for (int jj = 0; jj < JG; ++jj) {
      const int j = jg * JG + jj;
      const int nl = G::wave_n() * (JG * G::NB) + jj * G::NB + (G::lane() % G::NB);
#pragma unroll
      for (int i = 0; i < G::TM; ++i)
#pragma unroll
        for (int q = 0; q < G::VB / 4; ++q) {
          const f32x4_t v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *reinterpret_cast<f32x4_t*>(smem + nl * P + G::m_of(i, 4 * q) * 4) = v;
        }
    }
    lds_barrier();
    // Instruction i of a wave streams out the staged rows (wave + NWAVES i) RPI + h.  Their output row
    // indices are fetched once (lane RPW p + RPI i + h holds the one of phase p) and read back with
    // readlane, and the loop is unrolled in batches whose LDS reads are all issued before the first
    // store, so that a wave is not serialised on one LDS round trip per row.
    if (jg == 0) {
      const int l = G::lane();
      const int ph = l / RPW, idx = l % RPW;
      const int r = (G::wave() + G::NWAVES * (idx / RPI)) * RPI + idx % RPI;
      my_row = ph < NPH ? rows_lds[tile_col(ph, r)] : -1;
    }
    constexpr int RB = IPW < 8 ? IPW : 8;
#pragma unroll
    for (int i0 = 0; i0 < IPW; i0 += RB) {
      f32x4_t v[RB];
      int64_t orow[RB];
#pragma unroll
      for (int u = 0; u < RB; ++u)
        v[u] = *reinterpret_cast<const f32x4_t*>(smem + ((G::wave() + G::NWAVES * (i0 + u)) * RPI + h) * P + c * 16);
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        int64_t row = __builtin_amdgcn_readlane(my_row, jg * RPW + (i0 + u) * RPI);
#pragma unroll
        for (int hh = 1; hh < RPI; ++hh) {
          const int rh = __builtin_amdgcn_readlane(my_row, jg * RPW + (i0 + u) * RPI + hh);
          row = h == hh ? rh : row;
        }
        orow[u] = m < a.M ? row : -1;
      }
      if constexpr (Mode != 2) {
        if (accumulate) {
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            const OldT o = oldv[i0 + u];
            v[u] += f32x4_t{(float)o.x, (float)o.y, (float)o.z, (float)o.w};
          }
        }
      }
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int64_t row = orow[u];
        if (row < 0) continue;
        if (a.out_f) {
          *reinterpret_cast<f32x4_t*>(a.out_f + row * a.ldo + m) = v[u];
        } else if constexpr (ESZ == 4) {
          *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.out_e) + row * a.ldo + m) = v[u];
        } else {
          const bf16x4_t hb = {(__bf16)v[u].x, (__bf16)v[u].y, (__bf16)v[u].z, (__bf16)v[u].w};
          *reinterpret_cast<bf16x4_t*>(static_cast<__bf16*>(a.out_e) + row * a.ldo + m) = hb;
        }
      }
    }
    lds_barrier();
  }
}

// Tiles here are short (d_kv / 64 K-steps or fewer), so the workgroups are persistent: as many as
// are resident at a time (wg_per_cu of them on each compute unit), each taking every gridDim.x-th tile of the walk, which saves a workgroup
// launch per tile.  gridDim.x is a multiple of 8, so a tile stays on the XCD that the walk meant it for.
template <typename E, int Edge, int Mode, int Stages>
__global__ __launch_bounds__(256, wg_per_cu(Edge, Stages)) void kv_gemm_kernel(KvGemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (a.clear || (Mode == 2 && a.outside)) {
      int out = 0;
      if constexpr (Mode == 2)
        for (int g = 0; g < a.groups; ++g) out |= a.outside[g];
      a.hdr->err = out ? kErrKvCapacity : 0;
      a.hdr->nv = 0;
    }
  }
  for (int wg = blockIdx.x; wg < a.walk_len; wg += gridDim.x) kv_tile<E, Edge, Mode, Stages>(a, wg, smem);
}

// The end of a backward call: the workgroup's number says whether it takes 64 columns of db (a long chain of little work, so first; as
// many as keep the tiles on their XCDs), a tile of dW or of dU (the longer ones) or one of dx.  Bound by the tiles' K-steps where they
// fill the chip, by latency below.  4096 x 1024 in bf16: dx 13.7 us, both gradients 23.6, sums 9.9 in launches of their own; the whole
// call and its gate 145 us, with this 134.
template <typename E, int Edge>
__global__ __launch_bounds__(256, wg_per_cu(Edge, 0)) void kv_tail_kernel(KvGemmArgs dx, GemmTArgs g, KvSums q, int db_wgs, int grad_wgs) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int wg = blockIdx.x;
  if (wg < db_wgs) {
    if (wg >= q.d / 64) return;
    // four chains to a wavefront, added up in the order of kv_sum_kernel
    constexpr int kWaves = 4;
    float* const sm = reinterpret_cast<float*>(smem);
    const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6, j = wg * 64 + cl;
    column_sums<kSumWaves / kWaves>(q.dbpart + j, q.d, q.db_rows, rl, sm + rl * 64 + cl, kWaves * 64);
    __syncthreads();
    if (rl == 0) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < kSumWaves; ++w) v += sm[w * 64 + cl];
      q.db[j] = q.accumulate ? q.db[j] + v : v;
    }
    return;
  }
  wg -= db_wgs;
  if (wg < 2 * grad_wgs) {
    gemm_t_tile<E, 2, Edge, /*kSum=*/true>(g, wg < grad_wgs ? wg : wg - grad_wgs, wg >= grad_wgs, smem);
    return;
  }
  kv_tile<E, Edge, 3, 0>(dx, wg - 2 * grad_wgs, smem);
}

template <typename E, int Edge>
hipError_t launch_tail(const KvGemmArgs& dx, const GemmTArgs& g, const KvSums& q, hipStream_t s) {
  using G = KvTile<E, Edge, 3, 0>;
  static_assert(G::LDS_BYTES == Tile<E, false, Edge>::LDS_BYTES, "the two kinds of tiles share a workgroup's LDS");
  const int64_t mtiles = (dx.M + Edge - 1) / Edge, ntiles = (dx.Nn + Edge - 1) / Edge, side = (g.M + Edge - 1) / Edge;
  if (dx.out_f || !dx.out_e || dx.accumulate || dx.mode != 3 || !g.A2 || !g.done || g.ksplit < 1 || (g.ksplit > 1 && !g.part) ||
      (g.ksplit == 1 && g.part) || g.n_limit != g.M)
    return hipErrorInvalidValue;
  for (int64_t p : {g.ldA, g.ldB, g.ldB2})   // a K-step has to fit a window
    if (p > longest_pitch(1)) return hipErrorInvalidValue;
  KvGemmArgs b = dx;
  b.walk_len = (int)xcd_grid_size((int)mtiles, ntiles, kKvMapBy);
  const unsigned grad = xcd_grid_size((int)side, side * g.ksplit, kMapBy);
  hipError_t e = allow_lds<kv_tail_kernel<E, Edge>>(G::LDS_BYTES);
  if (e != hipSuccess) return e;
  const unsigned db = (unsigned)(q.d / 64 + kNumXcd - 1) / kNumXcd * kNumXcd;
  hipLaunchKernelGGL((kv_tail_kernel<E, Edge>), dim3(db + 2 * grad + (unsigned)b.walk_len), dim3(G::NT), G::LDS_BYTES, s, b, g, q, (int)db,
                     (int)grad);
  return hipGetLastError();
}

template <typename E, int Edge, int Mode, int Stages = 0>
hipError_t launch_tiles(const KvGemmArgs& a, hipStream_t s) {
  using G = KvTile<E, Edge, Mode, Stages>;
  const int mtiles = (a.M + G::BM - 1) / G::BM;
  const int64_t ntiles = (a.Nn + G::BN - 1) / G::BN;
  if (a.accumulate && (Mode == 2 || a.out_f || !a.out_e)) return hipErrorInvalidValue;
  KvGemmArgs b = a;
  b.walk_len = (int)xcd_grid_size(mtiles, ntiles, kKvMapBy);
  const unsigned resident = (unsigned)device_compute_units() / kNumXcd * kNumXcd * wg_per_cu(Edge, Stages);   // LDS-bound
  const dim3 grid(b.walk_len < (int)resident ? (unsigned)b.walk_len : resident);
  hipError_t e = allow_lds<kv_gemm_kernel<E, Edge, Mode, Stages>>(G::LDS_BYTES);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((kv_gemm_kernel<E, Edge, Mode, Stages>), grid, dim3(G::NT), G::LDS_BYTES, s, b);
  return hipGetLastError();
}

// ---- few tokens -----------------------------------------------------------------------------
//
// A decoding step's products (16 tokens x 1024 x 1024: 2 MB of parameters, 34 Mflop) are latency and nothing else.  One
// workgroup makes 16 tokens x 64 columns with sixteen wavefronts that share out the contraction, every load of a
// wavefront in flight at once, and the sixteen partial tiles are added up in LDS in a fixed order.  The
// parameter matrix is read as the caller has it, row k in memory = index k of the contraction: a lane takes 4
// consecutive columns of the rows it needs, so MFMA t of four covers the columns 4 r + t (r = MFMA row), and the
// bf16 fragments (8 values of k per lane and column) are put together with byte permutes.  kRows: out = x M^T, whose
// fragments lie in memory as they are; MFMA t covers the columns 16 t + r.  No transposed or padded copies, so the launch
// that made them goes too.
//
// kv_few_mask_kernel: the gate's logits, and their mask in the same launch.  The workgroups of 16 tokens count themselves, and the one
// that finishes last has the tokens' whole rows to read and a wavefront for each.  They come from workgroups on other XCDs, whose L2s do
// not see each other's lines: logits are stored and loaded at device scope, and the count goes up when a workgroup's stores
// have been acknowledged.  (Nobody waits for anybody.)
constexpr int kFewWaves = 16;

// The output of this thread: token threadIdx.x / kFewCols and column threadIdx.x % kFewCols of the workgroup's.
template <typename E, bool kRows>
__device__ inline float few_product(const KvFewArgs& a) {
  constexpr int PITCH = kFewCols + 4;   // floats
  __shared__ __attribute__((aligned(16))) float part[kFewWaves][kFewTok * PITCH];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int q = lane >> 4, tl = lane & 15;
  const int c0 = blockIdx.x * kFewCols, t0 = blockIdx.y * kFewTok;
  const int tok = min(t0 + tl, a.n - 1);   // tokens past the end re-read the last one
  f32x4_t acc[4] = {};
  const int nsub = a.d / 32;               // sub-steps of 32 values of k, dealt out to the wavefronts
  for (int s = w; s < nsub; s += kFewWaves) {
    if constexpr (Elem<E>::size == 2) {
      const char* const xp = static_cast<const char*>(a.x) + ((int64_t)tok * a.ldx + s * 32 + q * 8) * 2;
      const bf16x8_t fx = *reinterpret_cast<const bf16x8_t*>(xp);
      if constexpr (kRows) {
        const char* const mp = static_cast<const char*>(a.M) + ((int64_t)(c0 + tl) * a.d + s * 32 + q * 8) * 2;
        bf16x8_t f[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) f[t] = *reinterpret_cast<const bf16x8_t*>(mp + (int64_t)t * 16 * a.d * 2);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[t], fx, acc[t], 0, 0, 0);
      } else {
        const char* const mp = static_cast<const char*>(a.M) + ((int64_t)(s * 32 + q * 8) * a.d + c0 + tl * 4) * 2;
        uint2 row[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) row[e] = *reinterpret_cast<const uint2*>(mp + (int64_t)e * a.d * 2);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          u32x4_t f;
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const uint32_t lo = t < 2 ? row[2 * p].x : row[2 * p].y, hi = t < 2 ? row[2 * p + 1].x : row[2 * p + 1].y;
            f[p] = __builtin_amdgcn_perm(hi, lo, t & 1 ? 0x07060302u : 0x05040100u);
          }
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f), fx, acc[t], 0, 0, 0);
        }
      }
    } else {
      // one value of k per lane and MFMA: group q takes k = 32 s + 16 h + 4 q + e in MFMA e
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k0 = s * 32 + h * 16 + q * 4;
        const f32x4_t fx = *reinterpret_cast<const f32x4_t*>(static_cast<const float*>(a.x) + (int64_t)tok * a.ldx + k0);
        // rows[u]: four columns of row k0 + u, or (kRows) k0 .. k0 + 3 of column 16 u + tl
        const float* const mp = static_cast<const float*>(a.M) +
                                (kRows ? (int64_t)(c0 + tl) * a.d + k0 : (int64_t)k0 * a.d + c0 + tl * 4);
        f32x4_t rows[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) rows[u] = *reinterpret_cast<const f32x4_t*>(mp + (int64_t)(kRows ? 16 : 1) * u * a.d);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kRows ? rows[t][e] : rows[e][t], fx[e], acc[t], 0, 0, 0);
      }
    }
  }
  // accumulator v of MFMA t in lane group q is column 16 q + 4 v + t of the lane's token, or (kRows) 16 t + 4 q + v
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const f32x4_t o = kRows ? acc[u] : f32x4_t{acc[0][u], acc[1][u], acc[2][u], acc[3][u]};
    *reinterpret_cast<f32x4_t*>(&part[w][tl * PITCH + (kRows ? 16 * u + 4 * q : 16 * q + 4 * u)]) = o;
  }
  __syncthreads();
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < kFewWaves; ++u) sum += part[u][threadIdx.x / kFewCols * PITCH + threadIdx.x % kFewCols];
  return sum;
}

template <typename E>
using FewT = typename std::conditional<Elem<E>::size == 2, __bf16, float>::type;

template <typename E, bool kRows>
__global__ __launch_bounds__(64 * kFewWaves) void kv_few_kernel(KvFewArgs a) {
  if (a.hdr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    a.hdr->err = 0;
    a.hdr->nv = 0;
  }
  const float sum = few_product<E, kRows>(a);
  const int tok = blockIdx.y * kFewTok + threadIdx.x / kFewCols;
  if (tok >= a.n) return;
  if (a.clear && blockIdx.x == 0 && threadIdx.x == 0) a.clear[blockIdx.y] = 0;   // here: loads do not wait for the pointer
  const int64_t at = (int64_t)tok * a.d + blockIdx.x * kFewCols + threadIdx.x % kFewCols;
  if (a.flags & kFewWide) {
    static_cast<float*>(a.out)[at] = sum;
  } else {
    FewT<E>* const out = static_cast<FewT<E>*>(a.out) + at;
    *out = (FewT<E>)(a.flags & kFewAdd ? sum + (float)*out : sum);
  }
}

// NG: groups of 256 columns.
template <typename E, int NG>
__global__ __launch_bounds__(64 * kFewWaves) void kv_few_mask_kernel(KvFewArgs a, KvFewMask b) {
  using T = FewT<E>;
  const float sum = few_product<E, false>(a);
  const int t0 = blockIdx.y * kFewTok, tok = t0 + threadIdx.x / kFewCols;
  float* const logits = static_cast<float*>(a.out);
  if (tok < a.n)
    __hip_atomic_store(logits + (int64_t)tok * a.d + blockIdx.x * kFewCols + threadIdx.x % kFewCols, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __shared__ int last;
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(b.done + blockIdx.y, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.d / kFewCols - 1;
  __syncthreads();
  const int64_t mine = t0 + (threadIdx.x >> 6);
  if (!last || mine >= a.n) return;
  const float* const z = logits + mine * a.d;
  auto row4 = [&](int j) {
    const unsigned long long* const q = reinterpret_cast<const unsigned long long*>(z + j);
    const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float4(__builtin_bit_cast(float, (uint32_t)lo), __builtin_bit_cast(float, (uint32_t)(lo >> 32)),
                       __builtin_bit_cast(float, (uint32_t)hi), __builtin_bit_cast(float, (uint32_t)(hi >> 32)));
  };
  const int count = mask_token<T, NG>(row4, b.bias, static_cast<const T*>(b.xt), mine, a.d, b.tau, b.literal ? 1 : 0, b.m,
                                      static_cast<T*>(b.xhat));
  if ((threadIdx.x & 63) == 0) b.k[mine] = count;
}
static_assert(kFewTok * kFewCols == 64 * kFewWaves, "one output per thread");

template <typename E, int Mode>
hipError_t launch_mode(const KvGemmArgs& a, hipStream_t s) {
  const int cus = device_compute_units(), edge = kv_tile_edge(Elem<E>::size == 4, Mode, a.M, a.Nn, a.K, cus);
  if constexpr (Elem<E>::size == 2 && Elem<E>::block == 16) {
    if (kv_deep_tiles(Mode, edge, a.M, a.Nn, a.K, cus)) {
      if (edge == 64) return launch_tiles<E, 64, Mode, kStages>(a, s);
      if constexpr (Mode != 2) return launch_tiles<E, 128, Mode, kStages>(a, s);
    }
  }
  switch (edge) {
    case 64: return launch_tiles<E, 64, Mode>(a, s);
    case 128: return launch_tiles<E, 128, Mode>(a, s);
    default: return launch_tiles<E, 256, Mode>(a, s);
  }
}

template <typename E>
hipError_t launch_e(const KvGemmArgs& a, hipStream_t s) {
  switch (a.mode) {
    case 0: return launch_mode<E, 0>(a, s);
    case 1: return launch_mode<E, 1>(a, s);
    case 2: return launch_mode<E, 2>(a, s);
    default: return launch_mode<E, 3>(a, s);
  }
}

}  // namespace

hipError_t launch_kv_few(int dtype, const KvFewArgs& a, hipStream_t s, const KvFewMask* mask) {
  const dim3 grid((unsigned)(a.d / kFewCols), (unsigned)((a.n + kFewTok - 1) / kFewTok));
  const dim3 block(64 * kFewWaves);
  if (mask && (a.d > kKvFewMask || (a.flags & kFewRows) || !(a.flags & kFewWide) || !mask->k || !mask->done)) return hipErrorInvalidValue;
  auto typed = [&](auto tag) {
    using E = decltype(tag);
    if (!mask) {
      hipLaunchKernelGGL((a.flags & kFewRows ? kv_few_kernel<E, true> : kv_few_kernel<E, false>), grid, block, 0, s, a);
      return;
    }
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, a, *mask); };
    switch ((a.d + 255) / 256) {
      case 1: return launch(kv_few_mask_kernel<E, 1>);
      case 2: return launch(kv_few_mask_kernel<E, 2>);
      case 3: return launch(kv_few_mask_kernel<E, 3>);
      default: return launch(kv_few_mask_kernel<E, 4>);
    }
  };
  if (dtype == LMHEAD_BF16)
    typed(bf16_tag{});
  else
    typed(f32_tag{});
  return hipGetLastError();
}

hipError_t launch_kv_tail(int dtype, const KvGemmArgs& dx, const GemmTArgs& g, const KvSums& q, hipStream_t s) {
  if (dtype == LMHEAD_BF16) return g.edge == 64 ? launch_tail<bf16_tag, 64>(dx, g, q, s) : launch_tail<bf16_tag, 128>(dx, g, q, s);
  return g.edge == 64 ? launch_tail<f32_tag, 64>(dx, g, q, s) : hipErrorInvalidValue;
}

hipError_t launch_kv_gemm(int dtype, const KvGemmArgs& a, hipStream_t s) {
  return dtype == LMHEAD_BF16 ? launch_e<bf16_tag>(a, s) : launch_e<f32_tag>(a, s);
}

}  // namespace lmhead
