// The three MFMA kernels of the LM-head path, all built on GemmTile (gemm_core.h):
//   fwd_kernel    logits tile (vocabulary x tokens) -> max / sum-exp / sum-exp*z per token and tile,
//                 target-logit capture; nothing of the tile is stored           (log-softmax of L_CE, Eq. 9)
//   dz_kernel     logits tile recomputed -> dZ = g (onehot - softmax)
//   gemm_t_kernel plain contraction with a transposed, row-mapped fp32 store    (dH and dW)
// fwd_kernel and dz_kernel also exist for 8-bit (e4m3) copies of their operands.
//
// Orientation: the vocabulary (or d) runs along the MFMA M axis and tokens (or vocabulary
// rows of dW) along N.  With the MFMA accumulator layouts (16x16 blocks for bf16 and e4m3, 32x32 for
// fp32) a lane then owns ONE token column per block and 4 (or 16) vocabulary entries of it, so
// the softmax statistics are reduced inside the lane and need two (or one) cross-lane steps per
// tile; and a lane's four consecutive M entries are contiguous in the row-major outputs (dZ row,
// dH row, dW row).
#include <atomic>
#include <type_traits>

#include "common.h"
#include "gemm_t.h"
#include "logits_tile.h"

namespace lmhead {

namespace {

// Which operand leads the LDS ring in each kernel (see GemmTile::run); true = the B side.
// Measured on the 32x8x2048 workload with the 16x16x32 main loop: the logits kernels do best with the
// hidden states leading (+2 % and +1 % over W leading), the two backward contractions with the dZ side
// leading (within 0.5 % either way).
constexpr bool kLeadFwd = true, kLeadDz = true;

// The forward does best with narrower, taller blocks (measured on the 32x8x2048 workload).
constexpr int kFwdMapBx = 2, kFwdMapBy = 8;

template <typename E, int Edge>
__global__ __launch_bounds__(Tile<E>::NT, 256 / Edge) void fwd_kernel(FwdArgs a) {
  using G = Tile<E, kLeadFwd, Edge>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nv = a.hdr->nv;
  const int nblk = (nv + G::BN - 1) / G::BN;
  // one vocabulary tile x one token block per workgroup: short-lived workgroups are dispatched in
  // tile-walk order, which keeps the ones that share operand slabs in step with each other
  // a launch may cover several weight matrices over the same hidden states: the walk's x axis then
  // runs over (policy, vocabulary tile), and neighbours in x still share the token block's rows of Hc
  int tx, nb;
  if (!xcd_tile_coords(blockIdx.x, a.ntiles * a.npol, nblk, kFwdMapBx, kFwdMapBy, tx, nb)) return;
  trace_stamp(0, 1);
  const int pol = tx / a.ntiles;
  const int tile = tx - pol * a.ntiles;
  const char* Wp = static_cast<const char*>(a.W[0]);
#pragma unroll
  for (int p = 1; p < kMaxPolicies; ++p) Wp = (pol == p) ? static_cast<const char*>(a.W[p]) : Wp;
  float* const zy = a.zy + (size_t)pol * a.Ncap;
  int32_t* const gid = a.gid + (size_t)pol * a.Ncap;
  float* const part = a.part + (size_t)pol * 3 * a.ntiles * a.Ncap;
  const int64_t n0 = (int64_t)nb * G::BN;
  const int m0 = tile * G::BM;
  const int ksteps = a.d * Elem<E>::size / G::KB;
  const int64_t pitchH = a.ldHc * Elem<E>::size;
  const int64_t pitchW = a.ldW * Elem<E>::size;

  uint32_t offA[G::A_LD], offB[G::B_LD];
#pragma unroll
  for (int q = 0; q < G::A_LD; ++q) {
    const int row = G::ldA_row(q);
    offA[q] = (uint32_t)((min(m0 + row, a.V - 1) - m0) * pitchW) + G::ld_byte(row);
  }
#pragma unroll
  for (int q = 0; q < G::B_LD; ++q) {
    const int row = G::ldB_row(q);
    offB[q] = (uint32_t)(row * pitchH) + G::ld_byte(row);
  }
  // target ids of this lane's token columns: fetched before the main loop so that their latency is hidden
  int tkj[G::TN];
#pragma unroll
  for (int j = 0; j < G::TN; ++j) tkj[j] = a.tok_c[n0 + G::n_of(j)];

  typename G::Acc acc;
  G::zero(acc);
  trace_stamp(1, 1);
  G::run(acc, Wp + (int64_t)m0 * pitchW, offA, static_cast<const char*>(a.Hc) + n0 * pitchH, offB, ksteps, smem, 1);
  trace_stamp(2, 1); trace_cycles(2, 1);

  capture_target<G>(a, acc, tkj, m0, m0 + G::BM, n0, zy, gid);
  trace_stamp(11, 1);
  TileStats<G> stats;
  stats.clear();
  const bool want_t = a.want_entropy && pol == 0;   // entropy is reported for the first weight matrix only
  // vocabulary rows with m_const >= V - m0 - m_base are padding
  stats.add(acc, a.zscale, a.V - m0 - G::m_base(), m0 + G::BM <= a.V, want_t);
  trace_stamp(12, 1);
  float* red = reinterpret_cast<float*>(smem);  // [WGM][BN][3]
  stats.to_lds(red);
  trace_stamp(13, 1);
  stats.store(a, red, part, tile, n0, want_t);
#ifdef LMHEAD_TRACE
  trace_stamp(3, 1);
  trace_cycles(3, 1);
  if (g_trace && g_trace_kind == 1 && threadIdx.x == 0 && blockIdx.x < kTraceWorkgroups) {
    unsigned xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    unsigned long long* ids = g_trace + ((size_t)kTraceWorkgroups + blockIdx.x) * 16;   // next to the cycle counts
    ids[11] = __builtin_amdgcn_s_getreg(4 | (15 << 11));   // HW_ID, bits 15:0
    ids[12] = xcc;
    ids[13] = ((unsigned long long)tx << 32) | (unsigned)nb;
  }
#endif
}

template <typename E>
struct Store4;
template <>
struct Store4<bf16_tag> {
  __device__ static inline void row(void* p, float a, float b, float c, float d) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
    bf16x4_t v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
    *reinterpret_cast<bf16x4_t*>(p) = v;
  }
};
template <>
struct Store4<f32_tag> {
  __device__ static inline void row(void* p, float a, float b, float c, float d) {
    f32x4_t v = {a, b, c, d};
    *reinterpret_cast<f32x4_t*>(p) = v;
  }
};

// Row order of the W tile in LDS for the 16x16-block dZ kernel.  LDS row R = WM w + 16 i + r feeds
// row r of MFMA block i of wave row w (WM rows per wave row, a multiple of 32), and accumulator element v of lane
// group q belongs to block row r = 4 q + v.  Loading vocabulary row WM w + 32 (i / 2) + 8 q + 4 (i % 2) + v there makes
// the eight values that a lane holds in blocks 2a and 2a + 1 the vocabulary rows WM w + 32 a + 8 q + [0, 8) of its
// token: 16 bytes of a dZ row, stored straight from registers.
struct DzRows {
  __device__ static constexpr int tile_row_of_lds_row(int R) {
    return (R & ~31) + 8 * ((R >> 2) & 3) + 4 * ((R >> 4) & 1) + (R & 3);
  }
  // compile-time part of the tile row of element v of block i (the rest depends on the lane only)
  __device__ static constexpr int offset(int i, int v) { return 32 * (i >> 1) + 4 * (i & 1) + v; }
};

// Epilogue of the dZ kernel on 16x16 blocks with bf16 output (bf16 or e4m3 operands; permuted W rows):
// dZ = g (onehot - p) in bf16, token-major, straight from registers: 16 bytes per lane and block pair (a token's
// 64 contiguous bytes come from the four lane groups of one store).  dH and dW both read this one copy.
template <typename G>
__device__ inline void dz_epilogue_direct(const DzArgs& a, typename G::Acc& acc, int m0, int mrel0, int64_t n0) {
  typedef __attribute__((ext_vector_type(2))) float f32x2_t;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  static_assert(G::NB == 16 && G::VB == 4 && G::TM % 2 == 0, "pairs of blocks");
  const int q = G::lane() / 16;
  const int mb = G::wave_m() * G::WM + 8 * q;    // lane part of the tile-relative vocabulary row
  const int vlim = a.V - m0 - mb;                // vocabulary rows with offset >= vlim are padding
  const float kz = kLog2e * a.zscale;            // logit = accumulator * zscale

  // per-token scalars of this lane's token columns, requested in one batch (one exposed round trip per
  // tile; requested before the main loop they do not fit next to its double-buffered fragments, and the
  // compiler then spills each one right after its load, which serialises the loads)
  float gj[G::TN], lsej[G::TN];
  int relj[G::TN];
  bool hit = false;
#pragma unroll
  for (int j = 0; j < G::TN; ++j) {
    const int64_t n = n0 + G::n_of(j);
    gj[j] = a.g_c[n];
    lsej[j] = a.lse_c[n];
    relj[j] = a.tok_c[n];
  }
#pragma unroll
  for (int j = 0; j < G::TN; ++j) {
    hit |= (relj[j] >= m0) & (relj[j] < m0 + G::BM);
    relj[j] -= m0 + mb;                          // compared with compile-time constants
  }
  trace_stamp(11, 2);
  // mode 0: no target of the wave's columns in this tile, no padding rows: dZ = -g p, with |g| folded into
  //         the exponent and the sign applied to the packed pair.
  // mode 1: a target somewhere in the tile: the one-hot term by a select (about a third of the tiles have
  //         such a wave at V = 152 k).   mode 2: the vocabulary's last tile (padding rows give 0).
  const int mode = (m0 + G::BM <= a.V) ? (__any(hit) ? 1 : 0) : 2;
  char* const dZ = static_cast<char*>(a.dZ);

#pragma unroll
  for (int j = 0; j < G::TN; ++j) {
    const float g = gj[j];
    const float bias = -lsej[j] * kLog2e;
    const int rel = relj[j];
    const int tl = G::n_of(j);                   // token within the tile
    char* const grow = dZ + ((size_t)(n0 + tl) * a.ldZ + mrel0 + mb) * 2;
    auto emit = [&](auto mode_tag) {
      constexpr int kMode = decltype(mode_tag)::value;
      const float bias0 = bias + __builtin_amdgcn_logf(fabsf(g));   // log2 |g|; -inf for g = 0 gives p = 0
      const uint32_t smask = g > 0.f ? 0x80008000u : 0u;
      const float ng = -g;
#pragma unroll
      for (int ap = 0; ap < G::TM / 2; ++ap) {
        u32x4_t pk;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          float dz[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int i = 2 * ap + (w >> 1), v = 2 * (w & 1) + u;
            const float z = acc[i][j][v];
            if constexpr (kMode == 0) {
              dz[u] = fast_exp2(fmaf(z, kz, bias0));
            } else {
              const float p = fast_exp2(fmaf(z, kz, bias));
              const bool oh = DzRows::offset(i, v) == rel;
              if constexpr (kMode == 1)
                dz[u] = fmaf(ng, p, oh ? g : 0.f);
              else
                dz[u] = (DzRows::offset(i, v) < vlim) ? g * ((oh ? 1.f : 0.f) - p) : 0.f;
            }
          }
          const f32x2_t pair = {dz[0], dz[1]};
          uint32_t word = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2_t));
          if constexpr (kMode == 0) word ^= smask;
          pk[w] = word;
        }
        *reinterpret_cast<u32x4_t*>(grow + 64 * ap) = pk;
        __builtin_amdgcn_sched_barrier(0);        // one block pair's values live at a time
      }
    };
    if (mode == 0)
      emit(std::integral_constant<int, 0>{});
    else if (mode == 1)
      emit(std::integral_constant<int, 1>{});
    else
      emit(std::integral_constant<int, 2>{});
  }
}

// E: type of the operands Hc and W (possibly e4m3 copies); EO: type of dZ.
template <typename E, typename EO, int Edge>
__global__ __launch_bounds__(Tile<E>::NT, 256 / Edge) void dz_kernel(DzArgs a) {
  using G = Tile<E, kLeadDz, Edge>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nv = a.hdr->nv;
  const int nblk = (nv + G::BN - 1) / G::BN;
  int mt, nb;
  if (!xcd_tile_coords(blockIdx.x, a.ntiles * (kTile / Edge), nblk, kMapBx, kMapBy, mt, nb)) return;
  trace_stamp(0, 2);
  const int64_t n0 = (int64_t)nb * G::BN;
  const int mrel0 = mt * G::BM;  // within the chunk
  const int m0 = a.c0 + mrel0;
  if (m0 == 0) {
    const int64_t n = n0 + threadIdx.x;
    if (threadIdx.x < G::BN && n < nv && a.tok_c[n] < 0) atomicOr(&a.hdr->err, kErrTok);
  }
  const int mw = min(m0, a.V - 1);   // chunks end on multiples of 256: a narrower tile can lie beyond V (its dZ is 0)
  const int ksteps = a.d * Elem<E>::size / G::KB;
  const int64_t pitchH = a.ldHc * Elem<E>::size;
  const int64_t pitchW = a.ldW * Elem<E>::size;

  // With 16x16 blocks and bf16 output the rows of the W tile enter LDS in a permuted order (DzRows), chosen so that a
  // lane's accumulators of two neighbouring blocks are EIGHT consecutive vocabulary entries of its token:
  // 16 bytes of a dZ row, stored straight from registers.
  constexpr bool kDirect = G::NB == 16 && std::is_same<EO, bf16_tag>::value;
  uint32_t offA[G::A_LD], offB[G::B_LD];
#pragma unroll
  for (int q = 0; q < G::A_LD; ++q) {
    const int row = G::ldA_row(q);
    const int vrow = kDirect ? DzRows::tile_row_of_lds_row(row) : row;
    offA[q] = (uint32_t)((min(m0 + vrow, a.V - 1) - mw) * pitchW) + G::ld_byte(row);
  }
#pragma unroll
  for (int q = 0; q < G::B_LD; ++q) {
    const int row = G::ldB_row(q);
    offB[q] = (uint32_t)(row * pitchH) + G::ld_byte(row);
  }

  typename G::Acc acc;
  G::zero(acc);
  trace_stamp(1, 2);
  G::run(acc, static_cast<const char*>(a.W) + (int64_t)mw * pitchW, offA,
         static_cast<const char*>(a.Hc) + n0 * pitchH, offB, ksteps, smem, 2);
  trace_stamp(2, 2); trace_cycles(2, 2);
  if constexpr (kDirect) {
    dz_epilogue_direct<G>(a, acc, m0, mrel0, n0);
    trace_stamp(3, 2); trace_cycles(3, 2);
    return;
  }

  // Per-token scalars of this lane's token columns, requested after the main loop in one batch (one
  // exposed round trip per tile).  Requested before it they do not fit the register file next to the
  // loop's double-buffered fragments: the compiler then spills each one right after its load, which
  // serialises the loads (measured: a dozen dependent round trips per tile).
  float gj[G::TN], lsej[G::TN];
  int tkj[G::TN];
#pragma unroll
  for (int j = 0; j < G::TN; ++j) {
    const int64_t n = n0 + G::n_of(j);
    gj[j] = a.g_c[n];
    lsej[j] = a.lse_c[n];
    tkj[j] = a.tok_c[n];
  }
  float biasj[G::TN];
  int relj[G::TN];
  bool hit = false;
#pragma unroll
  for (int j = 0; j < G::TN; ++j) {
    biasj[j] = -lsej[j] * kLog2e;
    hit |= (tkj[j] >= m0) & (tkj[j] < m0 + G::BM);
    relj[j] = tkj[j] - m0 - G::m_base();   // compared with compile-time constants
  }

  char* dZ = static_cast<char*>(a.dZ);
  // The tile leaves through LDS so that it is written with full 16-byte-per-lane, line-contiguous stores: registers
  // hold 4 consecutive vocabulary entries of one token.  JG of the wave's TN token blocks are staged per phase.
  constexpr int ESZ = Elem<EO>::size;
  constexpr int JG0 = 64 / G::NB;
  constexpr int JG = JG0 < G::TN ? JG0 : G::TN;      // token blocks per wave per phase
  constexpr int NTOK = G::WGN * JG * G::NB;       // tokens staged per phase
  constexpr int P1 = G::BM * ESZ + 16;            // pitch of the [token][vocab] staging rows
  static_assert(NTOK * P1 <= G::LDS_BYTES, "staging fits in LDS");
  static_assert(G::TN % JG == 0, "phases cover the wave tile evenly");
  char* st1 = smem;
  const int vlim = a.V - m0 - G::m_base();
  const float kz = kLog2e * a.zscale;              // logit = accumulator * zscale
  // Which form of the element-wise work this wave needs (wave-uniform, see emit below).
  const int mode = (m0 + G::BM <= a.V) ? (__any(hit) ? 1 : 0) : 2;
#pragma unroll
  for (int jg = 0; jg < G::TN / JG; ++jg) {
#pragma unroll
    for (int jj = 0; jj < JG; ++jj) {
      const int j = jg * JG + jj;
      const float g = gj[j];
      const float bias = biasj[j];
      const int rel = relj[j];
      const int tl = G::wave_n() * (JG * G::NB) + jj * G::NB + (G::lane() % G::NB);   // token within the phase
      // mode 0: no target of the wave's columns in this tile, no padding rows: dZ = -g p.
      // mode 1: a target somewhere in the tile: the one-hot term by a select, still no tests around the
      //         exponential (about a third of the tiles have such a wave at V = 152 k).
      // mode 2: the vocabulary's last tile (padding rows give 0).
      auto emit = [&](auto mode_tag) {
        constexpr int kMode = decltype(mode_tag)::value;
        const float ng = -g;
#pragma unroll
        for (int i = 0; i < G::TM; ++i)
#pragma unroll
          for (int q = 0; q < G::VB / 4; ++q) {
            float dz[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float p = fast_exp2(fmaf(acc[i][j][4 * q + e], kz, bias));
              if constexpr (kMode == 0) {
                dz[e] = ng * p;
              } else if constexpr (kMode == 1) {
                dz[e] = fmaf(ng, p, (G::m_const(i, 4 * q + e) == rel) ? g : 0.f);
              } else {
                const float oh = (G::m_const(i, 4 * q + e) == rel) ? 1.f : 0.f;
                dz[e] = (G::m_const(i, 4 * q + e) < vlim) ? g * (oh - p) : 0.f;
              }
            }
            const int mt = G::m_of(i, 4 * q);   // tile-relative vocabulary row, multiple of 4
            Store4<EO>::row(st1 + tl * P1 + mt * ESZ, dz[0], dz[1], dz[2], dz[3]);
          }
      };
      if (mode == 0)
        emit(std::integral_constant<int, 0>{});
      else if (mode == 1)
        emit(std::integral_constant<int, 1>{});
      else
        emit(std::integral_constant<int, 2>{});
    }
    lds_barrier();
    // [token][vocab] rows -> dZ: one staged row is BM*ESZ contiguous bytes of a dZ row
    {
      constexpr int CPR = G::BM * ESZ / 16;   // 16-byte chunks per row
      constexpr int RPP = G::NT / CPR;        // rows per pass
      const int c = threadIdx.x % CPR;
#pragma unroll
      for (int r0 = 0; r0 < NTOK; r0 += RPP) {
        const int tl = r0 + threadIdx.x / CPR;
        const int nl = (tl / (JG * G::NB)) * G::WN + jg * (JG * G::NB) + tl % (JG * G::NB);   // token within the tile
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(st1 + tl * P1 + c * 16);
        *reinterpret_cast<u32x4_t*>(dZ + ((size_t)(n0 + nl) * a.ldZ + mrel0) * ESZ + c * 16) = v;
      }
    }
    if (jg + 1 < G::TN / JG) lds_barrier();
  }
}

// See gemm_t_tile; the role gives the uses distinct kernel names in profiles.
template <typename E, int Role, int Edge>
__global__ __launch_bounds__(Tile<E>::NT, 256 / Edge) void gemm_t_kernel(GemmTArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  gemm_t_tile<E, Role, Edge>(a, blockIdx.x, blockIdx.y != 0, smem);
}

}  // namespace

template <typename E, int Edge>
static hipError_t launch_fwd_e(const FwdArgs& a, hipStream_t s) {
  using G = Tile<E, false, Edge>;
  const dim3 grid(xcd_grid_size(a.ntiles * a.npol, a.Ncap / Edge, kFwdMapBy));
  hipError_t e = allow_lds<fwd_kernel<E, Edge>>(G::LDS_BYTES);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((fwd_kernel<E, Edge>), grid, dim3(G::NT), G::LDS_BYTES, s, a);
  return hipGetLastError();
}

template <typename E>
static hipError_t launch_fwd_edge(const FwdArgs& a, hipStream_t s) {
  switch (a.edge) {
    case 64: return launch_fwd_e<E, 64>(a, s);
    case 128: return launch_fwd_e<E, 128>(a, s);
    default: return launch_fwd_e<E, 256>(a, s);
  }
}

hipError_t launch_fwd(int dtype, const FwdArgs& a, hipStream_t s) {
  if (a.edge == 0) return launch_fwd_stream(a, s);
  if (dtype == kDtypeFp8) return launch_fwd_e<fp8_tag, 256>(a, s);   // its main loop is written for edge 256
  return dtype == LMHEAD_BF16 ? launch_fwd_edge<bf16_tag>(a, s) : launch_fwd_edge<f32_tag>(a, s);
}

template <typename E, typename EO, int Edge>
static hipError_t launch_dz_e(const DzArgs& a, hipStream_t s) {
  using G = Tile<E, false, Edge>;
  const dim3 grid(xcd_grid_size(a.ntiles * (kTile / Edge), a.Ncap / Edge, kMapBy));
  hipError_t e = allow_lds<dz_kernel<E, EO, Edge>>(G::LDS_BYTES);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((dz_kernel<E, EO, Edge>), grid, dim3(G::NT), G::LDS_BYTES, s, a);
  return hipGetLastError();
}

template <typename E>
static hipError_t launch_dz_edge(const DzArgs& a, hipStream_t s) {
  switch (a.edge) {
    case 64: return launch_dz_e<E, E, 64>(a, s);
    case 128: return launch_dz_e<E, E, 128>(a, s);
    default: return launch_dz_e<E, E, 256>(a, s);
  }
}

hipError_t launch_dz(int op_dtype, int out_dtype, const DzArgs& a, hipStream_t s) {
  if (op_dtype == kDtypeFp8)
    return out_dtype == LMHEAD_BF16 ? launch_dz_e<fp8_tag, bf16_tag, 256>(a, s) : launch_dz_e<fp8_tag, f32_tag, 256>(a, s);
  return op_dtype == LMHEAD_BF16 ? launch_dz_edge<bf16_tag>(a, s) : launch_dz_edge<f32_tag>(a, s);
}

template <typename E, int Role, int Edge>
static hipError_t launch_gemm_t_edge(const GemmTArgs& a, hipStream_t s) {
  using G = Tile<E, false, Edge>;
  const int64_t m_tiles = (a.M + Edge - 1) / Edge, n_cap = a.n_tiles_cap * (kTile / Edge);
  // slices chosen on the device: at most kSplitTiles slice tiles when there are several per tile
  const int64_t y_cap = a.ksplit > 0 ? n_cap * a.ksplit : (n_cap > kSplitTiles / m_tiles ? n_cap : kSplitTiles / m_tiles);
  const dim3 grid(xcd_grid_size((int)m_tiles, y_cap, kMapBy), a.A2 ? 2 : 1);
  hipError_t e = allow_lds<gemm_t_kernel<E, Role, Edge>>(G::LDS_BYTES);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_t_kernel<E, Role, Edge>), grid, dim3(G::NT), G::LDS_BYTES, s, a);
  return hipGetLastError();
}

template <typename E, int Role>
static hipError_t launch_gemm_t_impl(const GemmTArgs& a, hipStream_t s) {
  switch (a.edge) {
    case 64: return launch_gemm_t_edge<E, Role, 64>(a, s);
    case 128: return launch_gemm_t_edge<E, Role, 128>(a, s);
    default: return launch_gemm_t_edge<E, Role, 256>(a, s);
  }
}

hipError_t launch_gemm_t(int dtype, const GemmTArgs& a, hipStream_t s, int role) {
  if (role < 0) role = a.k_from_nv ? 1 : 0;
  int64_t pitch = a.ldA;   // of the K-major operands, whose K-step of 128 bytes of K has to fit a window
  if (role != 0)
    for (int64_t p : {a.ldB, a.A2 ? a.ldB2 : a.ldB}) pitch = p > pitch ? p : pitch;
  if (pitch > longest_pitch(1)) return hipErrorInvalidValue;
  if (dtype == LMHEAD_BF16)
    return role == 0   ? launch_gemm_t_impl<bf16_tag, 0>(a, s)
           : role == 1 ? launch_gemm_t_impl<bf16_tag, 1>(a, s)
                       : launch_gemm_t_impl<bf16_tag, 2>(a, s);
  return role == 0   ? launch_gemm_t_impl<f32_tag, 0>(a, s)
         : role == 1 ? launch_gemm_t_impl<f32_tag, 1>(a, s)
                     : launch_gemm_t_impl<f32_tag, 2>(a, s);
}

}  // namespace lmhead

#ifdef LMHEAD_TRACE
// Diagnostic build only (not part of the boundary): hands the kernel of the given kind (1 forward, 2 dZ, 3 dH,
// 4 dW) a device buffer of 2 x 2^19 x 16 64-bit words for its time stamps (see trace_stamp in gemm_core.h); NULL
// switches them off.
extern "C" __attribute__((visibility("default"))) int lmhead_debug_set_trace(void* dev_buf, int kind) {
  unsigned long long* p = static_cast<unsigned long long*>(dev_buf);
  hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(lmhead::g_trace_kind), &kind, sizeof(kind));
  if (e != hipSuccess) return (int)e;
  return (int)hipMemcpyToSymbol(HIP_SYMBOL(lmhead::g_trace), &p, sizeof(p));
}
#endif
