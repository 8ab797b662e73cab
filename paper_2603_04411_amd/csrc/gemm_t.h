// One tile of a plain contraction with a row-mapped fp32 store: dH and dW of the LM head, the parameter gradients of the KV gate.
#pragma once

#include <type_traits>

#include "common.h"
#include "gemm_core.h"

namespace lmhead {

namespace {

constexpr bool kLeadDh = true, kLeadDw = true;   // the dZ side leads the LDS ring

// Workgroup tile, four wavefronts (2 x 2).
template <typename E, bool kLeadB = false, int Edge = 256, bool kTransA = false, bool kTransB = false, bool kWalk = false>
using Tile = GemmTile<E, Edge, Edge, 2, 2, kLeadB, false, kTransA, kTransB, kWalk>;

// Block shape of the XCD-local tile walk (see xcd_tile_coords): 4 x 4 work items.
constexpr int kMapBx = 4, kMapBy = 4;
// Sixteen bytes that workgroups of one launch hand to each other, also across XCDs: at device scope (the sc1 bit), past the L2s, which
// do not see each other's lines.  base: the same in all lanes; at: bytes from it, below 2 GiB.
constexpr int kDeviceScope = 16;
__device__ inline __amdgpu_buffer_rsrc_t shared_window(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00020000);
}
__device__ inline void store_shared(__amdgpu_buffer_rsrc_t w, uint32_t at, f32x4_t v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), w, (int)at, 0, kDeviceScope);
}
__device__ inline f32x4_t load_shared(__amdgpu_buffer_rsrc_t w, uint32_t at) {
  return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(w, (int)at, 0, kDeviceScope));
}

// The operands that have the contraction along their rows are taken as they lie (GemmTile's K-major operands): W for
// dH, the hidden states and dZ for dW, both operands of a parameter gradient.  Against K-contiguous copies of all of them
// (8x8x256 step, d 2048, bf16): copies 294 -> 17 us (the zeroing of padding), dZ kernel, which had to write dZ in both orientations,
// 5.57 -> 5.01 ms, dH 4.46 -> 4.50, dW 4.48 -> 4.46, the step 19.7 -> 18.8 ms; 4x8x2048, d 4096: dZ 39.7 -> 38.0 ms (the
// step, 150 ms, by no more than its runs differ).  Which operand leads the ring makes no difference here; two transposing
// reads behind an MFMA instead of one cost dW 2 %.
// Role: 0 = dH (contracts over a vocabulary chunk), 1 = dW (contracts over the valid tokens), 2 = a
// parameter gradient of the KV gate (contracts over the tokens of a stream).  wg: position in the tile walk.  second: the second
// product of the launch (A2, B2).  kSum: the slices of a tile are added up by the last of its workgroups.
template <typename E, int Role, int Edge, bool kSum = false>
__device__ inline void gemm_t_tile(const GemmTArgs& a, int wg, bool second, char* smem) {
  constexpr bool kTB = Role != 0;
  using G = Tile<E, (Role == 0 ? kLeadDh : kLeadDw), Edge, /*kTransA=*/true, kTB, /*kWalk=*/Role == 1>;
  const int nv = a.hdr->nv;
  const int64_t n_lim = a.n_from_nv ? (int64_t)nv : a.n_limit;
  // the walk's y axis runs over (slice of the contraction, n tile): neighbours share the slice's K range
  const int ntiles = (int)((n_lim + G::BN - 1) / G::BN);
  const int ksplit = a.ksplit > 0 ? a.ksplit : a.hdr->ksplit;
  int mt, ny;
  if (!xcd_tile_coords(wg, (a.M + G::BM - 1) / G::BM, ntiles * ksplit, kMapBx, kMapBy, mt, ny)) return;
  // where the tile goes: a slice of the partial sums, or out
  const bool to_part = a.part && (a.ksplit > 0 || ksplit > 1 || a.part_single);
  const int slice = ny / ntiles;
  const int nt = ny - slice * ntiles;
  const int64_t n0 = (int64_t)nt * G::BN;
  const int m0 = mt * G::BM;
  const int64_t kel = a.k_from_nv ? (int64_t)nv : a.K;
  const int ksteps_all = (int)((kel * Elem<E>::size + G::KB - 1) / G::KB);
  const int per_slice = (ksteps_all + ksplit - 1) / ksplit;
  const int k_first = slice * per_slice;
  const int ksteps = max(0, min(per_slice, ksteps_all - k_first));
  const int64_t pitchA = a.ldA * Elem<E>::size;
  const int64_t pitchB = (second ? a.ldB2 : a.ldB) * Elem<E>::size;

  uint32_t offA[G::A_LD], offB[G::B_LD];
#pragma unroll
  for (int q = 0; q < G::A_LD; ++q) {
    const int row = G::ldT_row(q);
    offA[q] = (uint32_t)(row * pitchA) + G::ldT_byte(row);
  }
#pragma unroll
  for (int q = 0; q < G::B_LD; ++q) {
    const int row = kTB ? G::ldT_row(q) : G::ldB_row(q);
    offB[q] = (uint32_t)(row * pitchB) + (kTB ? G::ldT_byte(row) : G::ld_byte(row));
  }

  // The fp32 tile leaves through LDS as [n][m] rows, as many tile columns per phase as fit: CH lanes of 16 bytes per
  // row, RPI rows per wavefront instruction, RPW rows per wave and phase (rows wave, wave + 4, ... in units of RPI).
  // The output row that lane RPW p + RPI i + h needs in instruction i of phase p is fetched now; the epilogue reads
  // it with readlane instead of one dependent global load per row.
  constexpr int JG = 64 / G::NB < G::TN ? 64 / G::NB : G::TN;   // column blocks per wave per phase
  constexpr int NPH = G::TN / JG;
  constexpr int NCOL = G::WGN * JG * G::NB;       // tile columns (n) staged per phase
  constexpr int CH = G::BM * 4 / 16;              // lanes per staged row
  constexpr int RPI = 64 / CH;                    // staged rows per wavefront instruction
  constexpr int RPW = NCOL / G::NWAVES;           // staged rows per wave and phase
  constexpr int IPW = RPW / RPI;                  // instructions per wave and phase
  static_assert(G::TN % JG == 0 && 64 % CH == 0 && RPW % RPI == 0 && RPW * NPH <= 64, "one output row index per lane");
  int my_row = -1;
  {
    const int p = G::lane() / RPW, i = G::lane() % RPW;
    const int r = (G::wave() + G::NWAVES * (i / RPI)) * RPI + i % RPI;
    const int64_t n = n0 + (r / (JG * G::NB)) * G::WN + p * (JG * G::NB) + r % (JG * G::NB);
    if (p < NPH && n < n_lim) my_row = (int)(to_part ? n : (a.rowmap ? (int64_t)a.rowmap[n] : a.row_base + n));
  }
  const int64_t part_slice = a.ksplit > 0 ? a.part_slice : (int64_t)ntiles * G::BN * a.part_ld;
  float* const outp = to_part ? a.part + (size_t)(slice + (second ? ksplit : 0)) * part_slice : second ? a.out2 : a.out;
  const int64_t ldo = to_part ? a.part_ld : a.ldo;
  const bool accumulate = to_part ? a.part_accumulate : a.accumulate;

  typename G::Acc acc;
  G::zero(acc);
  constexpr int kKind = Role == 0 ? 3 : (Role == 1 ? 4 : 0);
  const char* const pa = static_cast<const char*>(second ? a.A2 : a.A);
  const char* const pb = static_cast<const char*>(second ? a.B2 : a.B);
  constexpr int ESZ = Elem<E>::size;
  if constexpr (Role == 1) {
    // both operands lie in the workspace and are readable to the end of their last K-step
    const int64_t stepA = G::KROWS * pitchA, stepB = G::KROWS * pitchB;
    G::run_steps(acc, pa + k_first * stepA + (int64_t)m0 * ESZ, offA, G::kWindow, (uint32_t)stepA,
                 pb + k_first * stepB + n0 * ESZ, offB, G::kWindow, (uint32_t)stepB, ksteps, smem, kKind);
  } else {
    // A K-major operand advances by KROWS of its rows per K-step.  What lies past its end (the rows that fill the last
    // K-step up) has to read as zeros: a buffer window does that, of at most 2 GiB; operands beyond that are taken in
    // pieces, each of which fills the pipeline anew (about a microsecond).
    const int64_t stepA = G::KROWS * pitchA, stepB = kTB ? G::KROWS * pitchB : (int64_t)G::KB;
    const int piece = window_ksteps(kTB && stepB > stepA ? stepB : stepA);   // at least one: launch_gemm_t
    const int64_t bytesA = second ? a.a2_bytes : a.a_bytes, bytesB = second ? a.b2_bytes : a.b_bytes;
    auto window = [](int64_t left) { return (uint32_t)(left < 0 ? 0 : left < G::kWindow ? left : G::kWindow); };
    int k = 0;
    do {
      const int64_t atA = (k_first + k) * stepA + (int64_t)m0 * ESZ;
      const int64_t atB = (k_first + k) * stepB + (kTB ? n0 * ESZ : n0 * pitchB);
      G::run_steps(acc, pa + atA, offA, window(bytesA - atA), (uint32_t)stepA, pb + atB, offB,
                   kTB ? window(bytesB - atB) : G::kWindow, (uint32_t)stepB, min(piece, ksteps - k), smem, kKind);
      k += piece;
    } while (k < ksteps);
  }

  // Rows go in batches: the LDS reads and the loads of the old values of a whole batch are issued before its
  // first store, so a wave that is alone on its SIMD does not sit out one memory round trip per row.
  constexpr int P = G::BM * 4 + 16;               // staging row pitch in bytes
  static_assert(NCOL * P <= G::LDS_BYTES, "staging fits in LDS");
  const int h = G::lane() / CH;                   // which of the instruction's rows this lane works on
  const int c = G::lane() % CH;                   // its 16-byte chunk of the row = 4 output columns
  const int m = m0 + c * 4;
  const bool m_ok = m < a.M;
  // dW is written once, gigabytes of it, and not read again by this library: past the caches, so that W, which the next
  // forward reads, can stay there in part (192 x 2048 x 151936: that forward 211 -> 185 us, the step 1177 -> 1152).  The
  // slices of a split contraction are read back at once and stay in (streamed too, dH took 199 us instead of 187), and
  // so does dW where the matrix cores bound it: over 5000 tokens or more streaming cost 0.1 to 0.4 % of the step.
  constexpr int64_t kStreamTokens = 2048;
  const bool stream = Role == 1 && !to_part && !accumulate && kel <= kStreamTokens;
#pragma unroll
  for (int jg = 0; jg < NPH; ++jg) {
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
    constexpr int RB = IPW < 8 ? IPW : 8;
#pragma unroll
    for (int i0 = 0; i0 < IPW; i0 += RB) {
      f32x4_t v[RB], old[RB];
      f32x4_t* dst[RB];
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        int64_t row = __builtin_amdgcn_readlane(my_row, jg * RPW + (i0 + u) * RPI);
#pragma unroll
        for (int hh = 1; hh < RPI; ++hh) {
          const int rh = __builtin_amdgcn_readlane(my_row, jg * RPW + (i0 + u) * RPI + hh);
          row = h == hh ? rh : row;
        }
        dst[u] = (row >= 0 && m_ok) ? reinterpret_cast<f32x4_t*>(outp + row * ldo + m) : nullptr;
        v[u] = *reinterpret_cast<const f32x4_t*>(smem + ((G::wave() + G::NWAVES * (i0 + u)) * RPI + h) * P + c * 16);
      }
      if (accumulate) {
#pragma unroll
        for (int u = 0; u < RB; ++u) old[u] = dst[u] ? *dst[u] : f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < RB; ++u) v[u] += old[u];
      }
      if (stream) {
#pragma unroll
        for (int u = 0; u < RB; ++u)
          if (dst[u]) __builtin_nontemporal_store(v[u], dst[u]);
      } else {
#pragma unroll
        for (int u = 0; u < RB; ++u)
          if (dst[u]) {
            if constexpr (kSum) {
              if (to_part) {
                store_shared(shared_window(outp), (uint32_t)((const char*)dst[u] - (const char*)outp), v[u]);
                continue;
              }
            }
            *dst[u] = v[u];
          }
      }
    }
    if (jg + 1 < NPH) lds_barrier();
  }
  if constexpr (kSum) {
    if (!to_part) return;
    // this workgroup's slice has arrived in memory; the one that finds all the others there adds them up, in their order
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* const last = reinterpret_cast<int*>(smem);
    const int mtiles = (a.M + G::BM - 1) / G::BM;
    if (threadIdx.x == 0)
      *last = __hip_atomic_fetch_add(a.done + ((second ? ntiles : 0) + nt) * mtiles + mt, 1, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT) == ksplit - 1;
    __syncthreads();
    if (!*last) return;
    constexpr int U = G::BM * G::BN / 4 / G::NT < 8 ? G::BM * G::BN / 4 / G::NT : 8;   // places of a thread whose slices are under way
    const float* const p0 = a.part + (size_t)(second ? ksplit : 0) * part_slice;
    float* const out = second ? a.out2 : a.out;
    for (int i0 = threadIdx.x; i0 < G::BN * CH; i0 += U * G::NT) {
      uint32_t at[U];
      bool in[U];
      f32x4_t t[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * G::NT;
        const int64_t n = n0 + i / CH;
        const int col = m0 + i % CH * 4;
        in[u] = n < n_lim && col < a.M;
        at[u] = in[u] ? (uint32_t)(n * a.part_ld + col) * 4 : 0;
        t[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
      for (int s = 0; s < ksplit; s += 4) {
        f32x4_t v[U][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const __amdgpu_buffer_rsrc_t w = shared_window(p0 + (size_t)min(s + e, ksplit - 1) * part_slice);
#pragma unroll
          for (int u = 0; u < U; ++u) v[u][e] = load_shared(w, at[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (s + e < ksplit) t[u] += v[u][e];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (in[u]) {
          const int i = i0 + u * G::NT;
          f32x4_t* const dst = reinterpret_cast<f32x4_t*>(out + (n0 + i / CH) * a.ldo + m0 + i % CH * 4);
          if (a.accumulate) t[u] += *dst;
          *dst = t[u];
        }
    }
  }
}

}  // namespace

}  // namespace lmhead
