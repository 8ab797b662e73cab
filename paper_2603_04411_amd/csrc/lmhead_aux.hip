// Bandwidth-bound helper kernels around the MFMA kernels: batch indexing (mask, prefix
// sums, compaction map), row gather of H and zero-filling of padded dH rows, 8-bit operand copies, the merge of
// the per-tile softmax statistics, the sum of split dH contractions.  All accesses are coalesced
// (16-byte vectors where rows allow); none of these kernels is more than a few passes
// over O(N d + V d) bytes.
#include <math.h>

#include <atomic>
#include <type_traits>

#include "common.h"

namespace lmhead {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// ---- indexing and gather of the valid rows ---------------------------------------------

// Header of a call: N_v, the error word (bad_len: a length outside [0, T]) and, with want_split, the cheapest allowed
// number of slices of dH's contraction (fewest on a tie): one wavefront, each lane prices one number.
__device__ inline void write_header(WsHeader* hdr, int nv, int bad_len, int want_split, const DhSplit& split, int lane) {
  if (want_split) {
    const int n_tiles = (nv + split.edge - 1) / split.edge;
    const int ks = lane + 1;
    static_assert(kMaxSplit == 64, "one number of slices per lane");
    const float cost = dh_split_allowed(split, n_tiles, ks) ? dh_split_cost(split, n_tiles, ks) : __builtin_huge_valf();
    float best = cost;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = fminf(best, __shfl_xor(best, o));
    const uint64_t ties = __ballot(cost == best);
    if (lane == 0) hdr->ksplit = __ffsll((unsigned long long)ties);
  }
  if (lane == 0) {
    hdr->nv = nv;
    hdr->err = bad_len ? kErrLen : 0;
  }
}

// Exclusive prefix sum of the clamped lengths by one workgroup of NT threads: out[0 .. R], out[R] = N_v; a
// length outside [0, T] sets `bad` in the thread that read it.  Ends with a barrier.
template <int NT>
__device__ inline void scan_lengths(const int32_t* __restrict__ len, int R, int T, int32_t* out, int& bad) {
  __shared__ int32_t wsum[NT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int carry = 0;
  for (int base = 0; base < R; base += NT) {
    const int r = base + tid;
    int x = 0;
    if (r < R) {
      x = len[r];
      if (x < 0 || x > T) {
        bad = 1;
        x = x < 0 ? 0 : T;
      }
    }
    int incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = carry;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      before += w < wave ? wsum[w] : 0;
      carry += wsum[w];
    }
    if (r < R) out[r] = before + incl - x;
    __syncthreads();
  }
  if (tid == 0) out[R] = carry;
  __syncthreads();
}

// Many responses: one workgroup scans the lengths and writes the header before the index kernel runs.
__global__ __launch_bounds__(1024) void scan_len_kernel(const int32_t* __restrict__ len, int R, int T,
                                                        WsHeader* hdr, int32_t* __restrict__ cu_ws,
                                                        int32_t* __restrict__ cu_out, int want_split, DhSplit split) {
  int bad = 0;
  scan_lengths<1024>(len, R, T, cu_ws, bad);
  bad = __syncthreads_or(bad);
  if (cu_out)
    for (int r = threadIdx.x; r <= R; r += 1024) cu_out[r] = cu_ws[r];
  if (threadIdx.x < 64) write_header(hdr, cu_ws[R], bad, want_split, split, threadIdx.x);
}

// Everything that the valid slots' positions decide, in one launch: mask, compaction map, and the gather of the
// valid rows of H (16 bytes per lane and step; zeros from N_v to the next tile multiple) with their token ids,
// gradients and statistics; for the backward the rows of dH of padded slots are zeroed.  Bound by the copy of H and the
// zeros.  kScan: each workgroup scans the lengths itself (up to kIndexMaxR of them, a microsecond), which saves the launch
// that would have to come first: three launches of 5 us each became one.  The range of the token ids is reported by the
// kernels that follow (an id outside [0, V) is -1 here): the header is only cleared in this launch.
// A wavefront takes kRows consecutive rows at a time; its lanes look up their slots together.  Four rows keep four loads in flight; up
// to kIndexFew slots there are not the wavefronts for that, and each takes one row, four chunks at a time (192 slots, d 2048: the
// scoring call 123 -> 120 us, the step 891 -> 883; 256 slots of fp32, d 256: the step 56.0 -> 55.2; from 8192 slots on no faster).
constexpr int kIndexMaxR = 4096, kIndexRows = 4, kIndexFew = 4096;
template <bool kScan, int kRows>
__global__ __launch_bounds__(256) void index_kernel(IndexArgs a) {
  __shared__ int32_t cu_s[kScan ? kIndexMaxR + 1 : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int32_t* cu = a.cu_ws;
  if constexpr (kScan) {
    int bad = 0;
    scan_lengths<256>(a.len, a.R, a.T, cu_s, bad);
    cu = cu_s;
    if (blockIdx.x == 0) {
      bad = __syncthreads_or(bad);
      for (int r = threadIdx.x; r <= a.R; r += 256) {
        a.cu_ws[r] = cu_s[r];
        if (a.cu_out) a.cu_out[r] = cu_s[r];
      }
      if (wave == 0) write_header(a.hdr, cu_s[a.R], bad, a.want_split, a.split, lane);
    }
  }
  const int64_t N = (int64_t)a.R * a.T;
  if (a.mask) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < N; i += (int64_t)gridDim.x * 256) {
      const int r = (int)(i / a.T);
      a.mask[i] = (int)(i - (int64_t)r * a.T) < cu[r + 1] - cu[r] ? 1 : 0;
    }
  }
  typedef __attribute__((ext_vector_type(4))) uint32_t u4;
  if (a.dH) {
    constexpr int PER = 4 * kRows;   // slots per wavefront and turn
    for (int64_t i0 = ((int64_t)blockIdx.x * 4 + wave) * PER; i0 < N; i0 += (int64_t)gridDim.x * 4 * PER) {
      const int64_t i = i0 + lane;
      bool pad = false;
      if (lane < PER && i < N) {
        const int r = (int)(i / a.T);
        pad = (int)(i - (int64_t)r * a.T) >= cu[r + 1] - cu[r];
      }
      for (uint64_t left = __ballot(pad); left; left &= left - 1) {
        u4* const row = reinterpret_cast<u4*>(a.dH + (i0 + __ffsll((unsigned long long)left) - 1) * a.dh_bytes);
        for (int64_t c = lane; c < a.dh_bytes / 16; c += 64) row[c] = u4{0, 0, 0, 0};
      }
    }
  }
  const int nv = cu[a.R];
  const int64_t nvp = ((int64_t)nv + kTile - 1) / kTile * kTile;
  const int nvec = a.row_bytes / 16;
  for (int64_t k0 = ((int64_t)blockIdx.x * 4 + wave) * kRows; k0 < nvp; k0 += (int64_t)gridDim.x * 4 * kRows) {
    // slot of row k0 + lane: the last response that starts at or before it (empty ones share their start with the next)
    const int64_t k = k0 + lane;
    int slot = -1;
    if (lane < kRows && k < nv) {
      int lo = 0, hi = a.R;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= k) lo = mid; else hi = mid;
      }
      slot = lo * a.T + (int)(k - cu[lo]);
    }
    if (lane < kRows) {
      a.row_slot[k] = slot;
      int tk = -1;
      if (slot >= 0) {
        tk = a.tok[slot];
        if (tk < 0 || tk >= a.V) tk = -1;
      }
      a.tok_c[k] = tk;
      if (a.g) a.g_c[k] = slot >= 0 ? a.g[slot] : 0.f;
      if (a.lse) a.lse_c[k] = slot >= 0 ? a.lse[slot] : 0.f;
      for (int p = 0; p < a.npol; ++p) {
        a.zy[p * a.Ncap + k] = 0.f;
        a.gid[p * a.Ncap + k] = -1;
      }
    }
    const u4* src[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      const int sl = __builtin_amdgcn_readlane(slot, u);
      src[u] = sl >= 0 ? reinterpret_cast<const u4*>(a.H + (int64_t)sl * a.pitchH) : nullptr;
    }
    constexpr int kAhead = kRows < 4 ? 4 / kRows : 1;   // chunks of a row on their way together
    for (int c = lane; c < nvec; c += 64 * kAhead) {
      u4 v[kRows][kAhead];
#pragma unroll
      for (int u = 0; u < kRows; ++u)
#pragma unroll
        for (int e = 0; e < kAhead; ++e) v[u][e] = src[u] && c + 64 * e < nvec ? src[u][c + 64 * e] : u4{0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < kRows; ++u)
#pragma unroll
        for (int e = 0; e < kAhead; ++e)
          if (c + 64 * e < nvec) reinterpret_cast<u4*>(a.Hc + (k0 + u) * a.pitchHc)[c + 64 * e] = v[u][e];
    }
  }
}
static_assert(kTile % kIndexRows == 0, "a wavefront's rows stay inside the padded extent");

// Eight (bf16) or four (fp32) values as e4m3: x * scale, rounded to nearest even.  The hardware conversion turns
// magnitudes beyond the format's range into NaN, so values are clamped to +-448 (the largest e4m3 number) first.
template <int N>
__device__ inline void to_e4m3(const float (&x)[N], float scale, uint32_t (&out)[N / 4]) {
  float v[N];
#pragma unroll
  for (int e = 0; e < N; ++e) v[e] = fminf(fmaxf(x[e] * scale, -448.f), 448.f);
#pragma unroll
  for (int w = 0; w < N / 4; ++w) {
    int p = 0;
    p = __builtin_amdgcn_cvt_pk_fp8_f32(v[4 * w], v[4 * w + 1], p, false);
    p = __builtin_amdgcn_cvt_pk_fp8_f32(v[4 * w + 2], v[4 * w + 3], p, true);
    out[w] = (uint32_t)p;
  }
}

// ---- 8-bit operand copies ---------------------------------------------------------------

// One wavefront per row: out = e4m3(in * scale), eight values per lane and pass.
template <typename T>
__global__ __launch_bounds__(256) void quantize_e4m3_kernel(const T* __restrict__ in, int64_t ld_in,
                                                            int64_t rows_fixed, int rows_from_nv,
                                                            const WsHeader* __restrict__ hdr, int cols,
                                                            float scale, uint8_t* __restrict__ out,
                                                            int64_t ld_out, int64_t rows_p) {
  const int64_t rows = rows_from_nv ? (int64_t)hdr->nv : rows_fixed;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows_p) return;
  if (rows_from_nv && r >= (rows + kTile - 1) / kTile * kTile) return;
  const int lane = threadIdx.x & 63;
  for (int c = lane * 8; c < cols; c += 512) {
    uint2 packed = make_uint2(0u, 0u);
    if (r < rows) {
      float v[8];
      if constexpr (sizeof(T) == 2) {
        typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
        const bf16x8 t = *reinterpret_cast<const bf16x8*>(in + r * ld_in + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (float)t[e];
      } else {
        const float4 t0 = *reinterpret_cast<const float4*>(in + r * ld_in + c);
        const float4 t1 = *reinterpret_cast<const float4*>(in + r * ld_in + c + 4);
        v[0] = t0.x; v[1] = t0.y; v[2] = t0.z; v[3] = t0.w;
        v[4] = t1.x; v[5] = t1.y; v[6] = t1.z; v[7] = t1.w;
      }
      uint32_t q[2];
      to_e4m3(v, scale, q);
      packed = make_uint2(q[0], q[1]);
    }
    *reinterpret_cast<uint2*>(out + r * ld_out + c) = packed;
  }
}

// ---- merge of per-tile softmax statistics ----------------------------------------------

// One workgroup per 64 slots (one per lane); its sixteen wavefronts each merge every sixteenth vocabulary tile,
// kFinBatch tiles at a time, and the sixteen results are merged in a fixed order.  The kernel reads
// 8 bytes (12 with entropy) per token and vocabulary tile once and is bound by those reads; what it has to avoid is a
// chain of dependent round trips: with one thread per slot and a serial loop over the tiles (two loops, in fact:
// maximum, then sums) it took 438 us for 120 tokens and 676 us for 41 k tokens at V = 151936 (0.3 TB/s), now 11 us
// and 58 us.  Sixteen wavefronts with 2 x 8 loads in flight each keep 64 KB per workgroup outstanding, enough
// for one workgroup per compute unit to run at memory speed when there are few tokens.
// Slots per workgroup: 64, one per lane.  Few slots, 16: the four quarters of a wavefront then merge tiles of their own
// with 64-byte reads (192 slots x 1187 tiles: 20.6 -> 13.2 us; 8192 slots x 594: 14.1 us with 64, 23.7 with 16).
// Also reports token ids that the index kernel found outside the vocabulary.
constexpr int kFinWaves = 16, kFinBatch = 8, kFinFewSlots = 2048;

// Statistics (m, s, t) of two disjoint sets of logits, scaled to the common maximum; exp2(-inf) = 0 drops empty ones.
__device__ inline void merge_stats(float& m, float& s, float& t, float m2, float s2, float t2) {
  const float mn = fmaxf(m, m2);
  const float ms = mn == -__builtin_huge_valf() ? 0.f : mn;
  const float f = __builtin_amdgcn_exp2f((m - ms) * kLog2e), f2 = __builtin_amdgcn_exp2f((m2 - ms) * kLog2e);
  s = s * f + s2 * f2;
  t = t * f + t2 * f2;
  m = mn;
}

template <int Slots>
__global__ __launch_bounds__(64 * kFinWaves) void finalize_kernel(const float* __restrict__ part,
                                                                  const float* __restrict__ zy,
                                                                  const int32_t* __restrict__ tok_c,
                                                                  WsHeader* __restrict__ hdr, int ntiles,
                                                                  int64_t Ncap, const int32_t* __restrict__ len,
                                                                  const int32_t* __restrict__ cu, int R, int T,
                                                                  float* __restrict__ logp, float* __restrict__ lse,
                                                                  float* __restrict__ ent) {
  constexpr int kStreams = kFinWaves * 64 / Slots;   // the tiles are dealt out to this many groups of Slots lanes
  __shared__ float red[kFinWaves][3][Slots];
  const int64_t N = (int64_t)R * T;
  const int lane = threadIdx.x % Slots, w = threadIdx.x / Slots;   // slot, stream
  const int64_t i = (int64_t)blockIdx.x * Slots + lane;
  int64_t k = -1;   // compact row of this slot, -1 on padding
  if (i < N) {
    const int r = (int)(i / T);
    const int t = (int)(i - (int64_t)r * T);
    if (t < min(max(len[r], 0), T)) k = cu[r] + t;
  }
  float m = -__builtin_huge_valf(), s = 0.f, tt = 0.f;
  if (k >= 0) {
    const size_t plane = (size_t)ntiles * Ncap;
    const float* const p = part + k;
    for (int c0 = w; c0 < ntiles; c0 += kStreams * kFinBatch) {
      float mc[kFinBatch], sc[kFinBatch], tc[kFinBatch];
#pragma unroll
      for (int u = 0; u < kFinBatch; ++u) {
        const int c = c0 + u * kStreams;
        const bool in = c < ntiles;
        mc[u] = in ? p[(size_t)c * Ncap] : -__builtin_huge_valf();
        sc[u] = in ? p[plane + (size_t)c * Ncap] : 0.f;
        tc[u] = in && ent ? p[2 * plane + (size_t)c * Ncap] : 0.f;
      }
      // a tile without a maximum holds nothing: its logits are all -inf, or NaN
#pragma unroll
      for (int u = 0; u < kFinBatch; ++u) {
        const bool none = mc[u] == -__builtin_huge_valf();
        sc[u] = none ? 0.f : sc[u];
        tc[u] = none ? 0.f : tc[u];
      }
      float mn = m;
#pragma unroll
      for (int u = 0; u < kFinBatch; ++u) mn = fmaxf(mn, mc[u]);
      const float ms = mn == -__builtin_huge_valf() ? 0.f : mn;
      const float old = __builtin_amdgcn_exp2f((m - ms) * kLog2e);
      s *= old;
      tt *= old;
#pragma unroll
      for (int u = 0; u < kFinBatch; ++u) {
        const float f = __builtin_amdgcn_exp2f((mc[u] - ms) * kLog2e);
        s = fmaf(sc[u], f, s);
        tt = fmaf(tc[u], f, tt);
      }
      m = mn;
    }
  }
  // the streams of a wavefront, then the wavefronts
#pragma unroll
  for (int o = Slots; o < 64; o <<= 1) {
    const float m2 = __shfl_xor(m, o), s2 = __shfl_xor(s, o), t2 = __shfl_xor(tt, o);
    merge_stats(m, s, tt, m2, s2, t2);
  }
  if (threadIdx.x % 64 < Slots) {
    red[threadIdx.x / 64][0][lane] = m;
    red[threadIdx.x / 64][1][lane] = s;
    red[threadIdx.x / 64][2][lane] = tt;
  }
  __syncthreads();
  if (w != 0 || i >= N) return;
  float o_lp = 0.f, o_lse = 0.f, o_ent = 0.f;
  if (k >= 0) {
    float mx = -__builtin_huge_valf();
#pragma unroll
    for (int q = 0; q < kFinWaves; ++q) mx = fmaxf(mx, red[q][0][lane]);
    const float ms = mx == -__builtin_huge_valf() ? 0.f : mx;
    s = 0.f;
    tt = 0.f;
#pragma unroll
    for (int q = 0; q < kFinWaves; ++q) {
      const float f = __builtin_amdgcn_exp2f((red[q][0][lane] - ms) * kLog2e);
      s = fmaf(red[q][1][lane], f, s);
      tt = fmaf(red[q][2][lane], f, tt);
    }
    o_lse = mx + __builtin_amdgcn_logf(s) * kLn2;
    o_lp = zy[k] - o_lse;
    o_ent = o_lse - tt / s;
    if (tok_c[k] < 0) atomicOr(&hdr->err, kErrTok);
  }
  logp[i] = o_lp;
  if (lse) lse[i] = o_lse;
  if (ent) ent[i] = o_ent;
}

// ---- sum of split contractions -----------------------------------------------------------

// One wavefront per 256 columns of a valid row n: out[rowmap(n)][:] (+)= part[0][n][:] + part[1][n][:] + ... (in this order), eight
// slices on their way at a time.  (One wavefront per row summed its columns one after the other, four slices at a time: 120 rows of
// 2048 columns 37 us, now 8.6; the step of 192 slots, d 2048, 880 -> 851 us, of 64 slots of d 768 313 -> 304.)
template <typename TO>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int ksplit,
                                                            int64_t part_slice, int64_t part_ld, int M,
                                                            const int32_t* __restrict__ rowmap,
                                                            const WsHeader* __restrict__ hdr, int64_t n_cap,
                                                            int64_t row_base, TO* __restrict__ out, int64_t ldo,
                                                            int accumulate, int edge, int single_too) {
  const int64_t n_valid = rowmap ? (int64_t)hdr->nv : n_cap;
  if (ksplit == 0) {
    ksplit = hdr->ksplit;
    if (ksplit == 1 && !single_too) return;
    part_slice = (n_valid + edge - 1) / edge * edge * part_ld;
  }
  const int lane = threadIdx.x & 63, chunks = (M + 255) / 256, waves = gridDim.x * 4;
  const int first = blockIdx.x * 4 + (threadIdx.x >> 6), rows_on = waves / chunks, chunks_on = waves - rows_on * chunks;
  int chunk = first % chunks;
  for (int64_t n = first / chunks; n < n_valid; n += rows_on) {
    const int64_t row = rowmap ? (int64_t)rowmap[n] : row_base + n;
    const int m = chunk * 256 + lane * 4;
    if (row >= 0 && m < M) {
      const float* const p = part + n * part_ld + m;
      float4 v = *reinterpret_cast<const float4*>(p);
      int s = 1;
      auto add = [&](auto count_tag) {
        constexpr int kCount = decltype(count_tag)::value;
        float4 q[kCount];
#pragma unroll
        for (int u = 0; u < kCount; ++u) q[u] = *reinterpret_cast<const float4*>(p + (size_t)(s + u) * part_slice);
#pragma unroll
        for (int u = 0; u < kCount; ++u) { v.x += q[u].x; v.y += q[u].y; v.z += q[u].z; v.w += q[u].w; }
        s += kCount;
      };
      while (s + 8 <= ksplit) add(std::integral_constant<int, 8>{});
      if (s + 4 <= ksplit) add(std::integral_constant<int, 4>{});
      if (s + 2 <= ksplit) add(std::integral_constant<int, 2>{});
      if (s < ksplit) add(std::integral_constant<int, 1>{});
      if constexpr (sizeof(TO) == 4) {
        float4* dst = reinterpret_cast<float4*>(out + row * ldo + m);
        if (accumulate) {
          const float4 o = *dst;
          v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
        }
        *dst = v;
      } else {
        typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
        const bf16x4_t h = {(__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
        *reinterpret_cast<bf16x4_t*>(out + row * ldo + m) = h;
      }
    }
    chunk += chunks_on;
    if (chunk >= chunks) {
      chunk -= chunks;
      ++n;
    }
  }
}

}  // namespace

hipError_t launch_index(const IndexArgs& a, hipStream_t s) {
  // one resident round of workgroups, or as many as there are rows and mask bytes for
  constexpr int64_t kMost = 2048;
  const int64_t cap = ((int64_t)a.R * a.T + kTile - 1) / kTile * kTile;
  const bool few = cap <= kIndexFew;
  const int64_t need = cap / (4 * (few ? 1 : kIndexRows));
  const dim3 grid((unsigned)(need < kMost ? need : kMost));
  if (a.R <= kIndexMaxR) {
    if (few)
      hipLaunchKernelGGL((index_kernel<true, 1>), grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((index_kernel<true, kIndexRows>), grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(scan_len_kernel, dim3(1), dim3(1024), 0, s, a.len, a.R, a.T, a.hdr, a.cu_ws, a.cu_out,
                       a.want_split, a.split);
    static_assert(kIndexFew <= kIndexMaxR, "so many responses are not few slots");
    hipLaunchKernelGGL((index_kernel<false, kIndexRows>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_quantize_e4m3(int dtype, const void* in, int64_t ld_in, int64_t rows_fixed, bool rows_from_nv,
                                const WsHeader* hdr, int cols, int exp2, void* out, int64_t ld_out, int64_t rows_p,
                                hipStream_t s) {
  const dim3 grid((unsigned)((rows_p + 3) / 4));
  const float scale = ldexpf(1.0f, exp2);
  if (dtype == LMHEAD_BF16)
    hipLaunchKernelGGL(quantize_e4m3_kernel<__bf16>, grid, dim3(256), 0, s, static_cast<const __bf16*>(in), ld_in,
                       rows_fixed, rows_from_nv ? 1 : 0, hdr, cols, scale, static_cast<uint8_t*>(out), ld_out, rows_p);
  else
    hipLaunchKernelGGL(quantize_e4m3_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(in), ld_in,
                       rows_fixed, rows_from_nv ? 1 : 0, hdr, cols, scale, static_cast<uint8_t*>(out), ld_out, rows_p);
  return hipGetLastError();
}

hipError_t launch_splitk_reduce(const float* part, int ksplit, int64_t part_slice, int64_t part_ld, int M,
                                const int32_t* rowmap, const WsHeader* hdr, int64_t n_cap, void* out, int64_t ldo,
                                bool accumulate, bool out_bf16, hipStream_t s, int64_t row_base, int edge,
                                bool single_too) {
  // rows are taken in turn by at most one resident round of workgroups: most of n_cap may turn out to be padding,
  // or the whole call idle
  constexpr int64_t kMost = 2048;
  const int64_t need = (n_cap * ((M + 255) / 256) + 3) / 4;
  const dim3 grid((unsigned)(need < kMost ? need : kMost));
  if (out_bf16)
    hipLaunchKernelGGL(splitk_reduce_kernel<__bf16>, grid, dim3(256), 0, s, part, ksplit, part_slice, part_ld, M,
                       rowmap, hdr, n_cap, row_base, static_cast<__bf16*>(out), ldo, 0, edge, single_too ? 1 : 0);
  else
    hipLaunchKernelGGL(splitk_reduce_kernel<float>, grid, dim3(256), 0, s, part, ksplit, part_slice, part_ld, M, rowmap,
                       hdr, n_cap, row_base, static_cast<float*>(out), ldo, accumulate ? 1 : 0, edge,
                       single_too ? 1 : 0);
  return hipGetLastError();
}

int device_compute_units() {
  constexpr int kMaxDev = 64;
  static std::atomic<int> cus[kMaxDev];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) return 256;
  int n = cus[dev].load(std::memory_order_acquire);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev].store(n, std::memory_order_release);
  }
  return n;
}

hipError_t launch_finalize(const float* part, const float* zy, const int32_t* tok_c, WsHeader* hdr, int ntiles,
                           int64_t Ncap, const int32_t* len, const int32_t* cu_len, int R, int T, float* logp,
                           float* lse, float* entropy, hipStream_t s) {
  const int64_t N = (int64_t)R * T;
  if (N <= kFinFewSlots)
    hipLaunchKernelGGL(finalize_kernel<16>, dim3((unsigned)((N + 15) / 16)), dim3(64 * kFinWaves), 0, s, part, zy, tok_c,
                       hdr, ntiles, Ncap, len, cu_len, R, T, logp, lse, entropy);
  else
    hipLaunchKernelGGL(finalize_kernel<64>, dim3((unsigned)((N + 63) / 64)), dim3(64 * kFinWaves), 0, s, part, zy, tok_c,
                       hdr, ntiles, Ncap, len, cu_len, R, T, logp, lse, entropy);
  return hipGetLastError();
}

}  // namespace lmhead
