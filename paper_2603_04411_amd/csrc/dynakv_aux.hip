// Bandwidth-bound kernels of the KV-compression path: the truncation mask (softmax, cumulative
// sum, threshold; Eqs. 5-8), the ragged store (offset scan + segment copy), the grouping of
// tokens by contraction length for the reconstruction, and the retain rate (Eqs. 4 and 9).
// Rows are handled one wavefront per token with 16-byte accesses.
#include "dynakv_mask.h"

namespace lmhead {

namespace {

// First write of every call to the error word (and the token count, which this path does not use).
__device__ inline void clear_header(WsHeader* hdr) {
  hdr->err = 0;
  hdr->nv = 0;
}

// ---- truncation mask -----------------------------------------------------------------------
//
// One wavefront per token (mask_token).
template <typename T, int NG>
__global__ __launch_bounds__(256) void kv_mask_kernel(const float* __restrict__ logits,
                                                      const float* __restrict__ bias,
                                                      const T* __restrict__ xt, int64_t n, int d, float tau,
                                                      int literal, int32_t* __restrict__ k_out,
                                                      float* __restrict__ m_out, T* __restrict__ xhat) {
  const int64_t tok = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tok >= n) return;
  const float* z = logits + tok * d;
  const int count = mask_token<T, NG>([&](int j) { return *reinterpret_cast<const float4*>(z + j); }, bias, xt, tok, d, tau, literal,
                                      m_out, xhat);
  if ((threadIdx.x & 63) == 0) k_out[tok] = count;
}

// ---- backward of the truncation mask ---------------------------------------------------------
//
// Chain rule through Eqs. 5-7 for one token, in the position order of kv_mask_kernel (position i =
// component i of x~, x^ and m; gate column j(i) = i, or d-1-i for Eq. 6 as printed):
//   p_i = softmax of the logits (+ bias),   m_i = sum_{i' >= i} p_i'          (recomputed)
//   q_i = dL/dm_i  = g_xhat_i * x~_i + g_m_i + g_m_const
//   r_i = dL/dp_i  = sum_{i' <= i} q_i'                (p_i feeds m_0 .. m_i)
//   g_l = dL/dlogit at column j(i) = p_i * (r_i - sum_i' p_i' r_i')             (softmax Jacobian)
//   a_i = g_xhat_i * m_i                               (the direct part of dL/dx~)
// One wavefront per token, looping over tokens with the grid's stride.  Each wavefront adds its g_l
// rows into its own strip of LDS (a lane always owns the same positions, so no atomics and a fixed
// order); the workgroup's four strips are summed at the end into one row of dbpart.
// NG as in kv_mask_kernel: NG > 0 keeps the row and q (then r) in registers; NG == 0 re-reads.
// Up to d = 1024 the kernel is held to 128 VGPRs so that four workgroups share a compute unit.
template <typename T, int NG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NG > 0 && NG <= 4 ? 4 : 2)))
void kv_mask_bwd_kernel(const float* __restrict__ logits, const float* __restrict__ bias, const T* __restrict__ xt,
                        const T* __restrict__ gxh, const float* __restrict__ gm, float gmc, int64_t n, int d,
                        int literal, T* __restrict__ gl, T* __restrict__ a_out, float* __restrict__ dbpart, int32_t* __restrict__ clear,
                        int nclear) {
  extern __shared__ float colsum[];   // [4][d], position order
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < nclear; i += 256) clear[i] = 0;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  float* const acc = colsum + wave * d;
  const int ngroups = NG > 0 ? NG : (d + 255) / 256;
  for (int g = 0; g < ngroups; ++g) {
    const int i0 = g * 256 + lane * 4;
    if (i0 < d) *reinterpret_cast<float4*>(acc + i0) = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  constexpr int NR = NG > 0 ? NG : 1;

  for (int64_t tok = (int64_t)blockIdx.x * 4 + wave; tok < n; tok += (int64_t)gridDim.x * 4) {
    const float* z = logits + tok * d;
    auto load4 = [&](int i0, float (&v)[4]) {
      if (!literal) {
        const float4 a = *reinterpret_cast<const float4*>(z + i0);
        const float4 b = *reinterpret_cast<const float4*>(bias + i0);
        v[0] = a.x + b.x; v[1] = a.y + b.y; v[2] = a.z + b.z; v[3] = a.w + b.w;
      } else {
        const int j0 = d - 4 - i0;
        const float4 a = *reinterpret_cast<const float4*>(z + j0);
        const float4 b = *reinterpret_cast<const float4*>(bias + j0);
        v[0] = a.w + b.w; v[1] = a.z + b.z; v[2] = a.y + b.y; v[3] = a.x + b.x;
      }
    };

    // softmax statistics, as in the forward kernel
    float row[NR][4];
    float mx = -__builtin_huge_valf();
    float sum = 0.f;
    if constexpr (NG > 0) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int i0 = g * 256 + lane * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) row[g][e] = -__builtin_huge_valf();
        if (i0 < d) load4(i0, row[g]);
      }
#pragma unroll
      for (int g = 0; g < NG; ++g) mx = fmaxf(fmaxf(mx, fmaxf(row[g][0], row[g][1])), fmaxf(row[g][2], row[g][3]));
      mx = wave_max(mx);
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          row[g][e] = __builtin_amdgcn_exp2f((row[g][e] - mx) * kLog2e);
          sum += row[g][e];
        }
    } else {
      for (int g = 0; g < ngroups; ++g) {
        const int i0 = g * 256 + lane * 4;
        if (i0 < d) {
          float v[4];
          load4(i0, v);
          mx = fmaxf(fmaxf(mx, fmaxf(v[0], v[1])), fmaxf(v[2], v[3]));
        }
      }
      mx = wave_max(mx);
      for (int g = 0; g < ngroups; ++g) {
        const int i0 = g * 256 + lane * 4;
        if (i0 < d) {
          float v[4];
          load4(i0, v);
#pragma unroll
          for (int e = 0; e < 4; ++e) sum += __builtin_amdgcn_exp2f((v[e] - mx) * kLog2e);
        }
      }
    }
    sum = wave_sum(sum);
    const float inv = 1.0f / sum;

    // the lane's four exponentials of group g (0 beyond d)
    auto expo = [&](int g, float (&s)[4]) {
      if constexpr (NG > 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = row[g][e];
      } else {
        const int i0 = g * 256 + lane * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = 0.f;
        if (i0 < d) {
          float v[4];
          load4(i0, v);
#pragma unroll
          for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_exp2f((v[e] - mx) * kLog2e);
        }
      }
    };
    // q of group g (0 beyond d) and the g_xhat values it was formed from
    auto load_q = [&](int g, float (&q)[4], float (&gx)[4]) {
      const int i0 = g * 256 + lane * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] = gx[e] = 0.f;
      if (i0 < d) {
        float xv[4];
        Store4<T>::load(xt + tok * d + i0, xv);
        Store4<T>::load(gxh + tok * d + i0, gx);
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = gx[e] * xv[e] + gmc;
        if (gm) {
          const float4 t = *reinterpret_cast<const float4*>(gm + tok * d + i0);
          q[0] += t.x; q[1] += t.y; q[2] += t.z; q[3] += t.w;
        }
      }
    };
    // q of one group turned, in place, into r: the inclusive prefix sums over all positions up to each one
    auto scan_prefix = [&](float& carry, float (&r)[4]) {
      r[1] += r[0];
      r[2] += r[1];
      r[3] += r[2];
      float incl = r[3];
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const float y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
      }
      const float below = carry + (incl - r[3]);
      carry += __shfl(incl, 63);
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] += below;
    };

    // m (suffix sums, last group first), a = g_xhat * m, and q (kept when the row is held in registers)
    float qk[NR][4];
    {
      float carry = 0.f;
      auto step = [&](int g, float (&q)[4]) {
        const int i0 = g * 256 + lane * 4;
        float sfx[4];
        expo(g, sfx);
        sfx[2] += sfx[3];
        sfx[1] += sfx[2];
        sfx[0] += sfx[1];
        float incl = sfx[0];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const float y = __shfl_down(incl, o);
          if (lane + o < 64) incl += y;
        }
        const float above = carry + (incl - sfx[0]);
        carry += __shfl(incl, 0);
        float gx[4];
        load_q(g, q, gx);
        if (i0 < d) {
#pragma unroll
          for (int e = 0; e < 4; ++e) gx[e] *= (above + sfx[e]) * inv;
          Store4<T>::store(a_out + tok * d + i0, gx);
        }
      };
      if constexpr (NG > 0) {
#pragma unroll
        for (int g = NG - 1; g >= 0; --g) step(g, qk[g]);
      } else {
        for (int g = ngroups - 1; g >= 0; --g) step(g, qk[0]);
      }
    }

    // r (in place of q) and s = sum_i p_i r_i
    float s = 0.f;
    {
      float carry = 0.f;
      auto step = [&](int g, float (&r)[4]) {
        if constexpr (NG == 0) {
          float gx[4];
          load_q(g, r, gx);
        }
        scan_prefix(carry, r);
        float ex[4];
        expo(g, ex);
#pragma unroll
        for (int e = 0; e < 4; ++e) s += ex[e] * r[e];
      };
      if constexpr (NG > 0) {
#pragma unroll
        for (int g = 0; g < NG; ++g) step(g, qk[g]);
      } else {
        for (int g = 0; g < ngroups; ++g) step(g, qk[0]);
      }
    }
    s = wave_sum(s) * inv;

    // g_l = p (r - s), stored in gate column order and added to the wavefront's column sums
    {
      float carry = 0.f;
      auto step = [&](int g, float (&r)[4]) {
        const int i0 = g * 256 + lane * 4;
        if constexpr (NG == 0) {
          float gx[4];
          load_q(g, r, gx);
          scan_prefix(carry, r);
        }
        float ex[4];
        expo(g, ex);
        if (i0 < d) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = ex[e] * inv * (r[e] - s);
          float4 t = *reinterpret_cast<const float4*>(acc + i0);
          t.x += v[0]; t.y += v[1]; t.z += v[2]; t.w += v[3];
          *reinterpret_cast<float4*>(acc + i0) = t;
          if (!literal) {
            Store4<T>::store(gl + tok * d + i0, v);
          } else {
            const float w[4] = {v[3], v[2], v[1], v[0]};
            Store4<T>::store(gl + tok * d + (d - 4 - i0), w);
          }
        }
      };
      if constexpr (NG > 0) {
#pragma unroll
        for (int g = 0; g < NG; ++g) step(g, qk[g]);
      } else {
        for (int g = 0; g < ngroups; ++g) step(g, qk[0]);
      }
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < d; c += 256) {
    const float t = ((colsum[c] + colsum[d + c]) + colsum[2 * d + c]) + colsum[3 * d + c];
    dbpart[(int64_t)blockIdx.x * d + (literal ? d - 1 - c : c)] = t;
  }
}

// The sums that end a backward call, in one launch: the slices of the two parameter gradients (if they were cut) and the
// column sums of the mask backward.  Bound by reading the parts once; what differs is where the parallelism is.
//  - Slices (few rows, d x d columns): one thread per four columns walks the rows.
//  - Column sums (many rows, d columns): a workgroup owns 64 columns, its sixteen wavefronts each sum every sixteenth
//    row, eight loads at a time.  (With four wavefronts and a chain of four loads each, 1024 rows of 1024 columns took 22 us, now 5.4.)
//    The slices of small parameters (d up to kSumByColumns) are as many as 256 and a thread per four columns would be two to eight
//    workgroups: they are summed like this too.  Whole backward call, us, by threads / by columns: bf16 40000 x 64 95.0 / 58.6
//    12000 x 128 46.9 / 40.1   fp32 12000 x 64 66.7 / 40.1;   not at d 256: 12000 x 256 49.0 / 51.3.
// The column sums are ready long before the gradients, but a launch of their own costs its 4 us of dispatch wherever it is put
// (4096 x 1024 training pair 149.5 -> 145.7 us; 300 x 128 in fp32 48.5 -> 47.4 with the one-launch retain rate below, which
// no longer waits for the GPU but for the host).
constexpr int kSumByColumns = 128;

__device__ inline void sum_slices(const float* __restrict__ part, int rows, int64_t row_pitch, float* __restrict__ out,
                                  int64_t j, bool accumulate) {
  float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int r = 0; r < rows; ++r) {
    const float4 v = reinterpret_cast<const float4*>(part + (int64_t)r * row_pitch)[j];
    t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
  }
  float4* const dst = reinterpret_cast<float4*>(out) + j;
  if (accumulate) {
    const float4 o = *dst;
    t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
  }
  *dst = t;
}

__global__ __launch_bounds__(64 * kSumWaves) void kv_sum_kernel(KvSums a, int by_columns) {
  __shared__ float sm[kSumWaves][64];
  const int col_blocks = a.d / 64;
  const int64_t len = (int64_t)a.d * a.d;
  const float* part = a.dbpart;
  float* out = a.db;
  int64_t rows = a.db_rows, pitch = a.d, j0 = (int64_t)blockIdx.x * 64;
  if ((int)blockIdx.x >= col_blocks) {
    const int64_t at = (int64_t)(blockIdx.x - col_blocks) * (by_columns ? 64 : 4 * 64 * kSumWaves);
    if (!by_columns) {
      int64_t j = at / 4 + threadIdx.x;
      const bool second = j >= len / 4;
      if (second) j -= len / 4;
      if (j < len / 4) sum_slices(a.part + (second ? a.slices * len : 0), a.slices, len, second ? a.dU : a.dW, j, a.accumulate);
      return;
    }
    const bool second = at >= len;
    part = a.part + (second ? a.slices * len : 0);
    out = second ? a.dU : a.dW;
    rows = a.slices;
    pitch = len;
    j0 = second ? at - len : at;
  }
  const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
  const int64_t j = j0 + cl;
  column_sums<1>(part + j, pitch, rows, rl, &sm[rl][cl], 0);
  __syncthreads();
  if (rl == 0) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kSumWaves; ++w) v += sm[w][cl];
    out[j] = a.accumulate ? out[j] + v : v;
  }
}

// ---- operand copies, with what else a call has to prepare ------------------------------------

__device__ inline int bucket_of(int k, int d, int esz) {
  k = min(max(k, 0), d);
  return (k * esz + 127) / 128;
}

// One launch prepares a call: it clears the header, puts the parameter matrices of the one-kernel gate into fragment order
// (64 x 64 tiles through LDS, 16-byte accesses on both sides) and counts the tokens of each length for the reconstruction's
// grouping.  Every one of these was a launch of its own, 3-5 us each and mostly dispatch.
__global__ __launch_bounds__(256) void kv_prepare_kernel(KvPrepareArgs a, int esz) {
  constexpr int VEC = 8;         // elements per 16-byte chunk
  constexpr int CPR = 64 / VEC;  // chunks per tile row
  constexpr int PITCH = 66;      // elements; keeps rows 4-byte aligned and the gather conflict-free
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * PITCH];
  if (a.hdr && blockIdx.x == 0 && threadIdx.x == 0) clear_header(a.hdr);
  int b = blockIdx.x;
  if (b < a.count.blocks) {
    // counts per K-step bucket of this block's tokens; no global atomics, so nothing has to be cleared first
    int32_t* const h = reinterpret_cast<int32_t*>(tile);   // nbuckets <= 257
    for (int i = threadIdx.x; i < a.count.nbuckets; i += 256) h[i] = 0;
    __syncthreads();
    const int64_t t1 = min(a.count.n, (int64_t)(b + 1) * a.count.per_block);
    for (int64_t i = (int64_t)b * a.count.per_block + threadIdx.x; i < t1; i += 256)
      atomicAdd(&h[bucket_of(a.count.k[i], a.count.d, esz)], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < a.count.nbuckets; i += 256) a.count.hist[(int64_t)b * a.count.nbuckets + i] = h[i];
    return;
  }
  if (a.njobs == 0) return;
  b -= a.count.blocks;
  const int row_tiles = a.job[0].d / 64, tiles = row_tiles * row_tiles;   // the jobs' matrices are of one size
  const KvCopy& c = a.job[b < tiles ? 0 : 1];
  if (b >= tiles) b -= tiles;
  const int d = c.d;
  const uint16_t* const in = static_cast<const uint16_t*>(c.in);
  uint16_t* const out = static_cast<uint16_t*>(c.out);
  const int r0 = b % row_tiles * 64, c0 = b / row_tiles * 64;
#pragma unroll
  for (int pass = 0; pass < 64 * CPR / 256; ++pass) {
    const int id = pass * 256 + threadIdx.x;
    const int rr = id / CPR, cc = id % CPR;
    const uint4 v = *reinterpret_cast<const uint4*>(in + (int64_t)(r0 + rr) * d + c0 + cc * VEC);
    uint32_t* const dst = reinterpret_cast<uint32_t*>(tile + rr * PITCH + cc * VEC);
    dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
  }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < 64 * CPR / 256; ++pass) {
    const int id = pass * 256 + threadIdx.x;
    const int col = id / CPR, rc = id % CPR;
    uint16_t e[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) e[i] = tile[(rc * VEC + i) * PITCH + col];
    uint4 v;
    __builtin_memcpy(&v, e, 16);
    const int k = r0 + rc * VEC;
    const int pos = c.flipped ? d - 1 - (c0 + col) : c0 + col;
    constexpr int NW = kKvGateWaves;
    const int w = pos / (d / NW), q = pos % (d / NW) / (d / (4 * NW)), i = pos % (d / (4 * NW)) / 4;
    const int lane = k / 8 % 4 * 16 + 4 * q + pos % 4;
    *reinterpret_cast<uint4*>(out + (((int64_t)w * (d / 32) + k / 32) * (d / (16 * NW)) + i) * 512 + lane * 8) = v;
  }
}

// ---- ragged store ---------------------------------------------------------------------------

__device__ inline int seg_len(int k, int d, int& bad) {
  if (k < 0 || k > d) {
    bad = 1;
    k = k < 0 ? 0 : d;
  }
  return (k + DYNAKV_GRANULE - 1) / DYNAKV_GRANULE * DYNAKV_GRANULE;
}

// Block totals of the segment lengths (kKvScanBlock tokens per block).  Clears the header: the counts are checked, and
// errors raised, by the kernel that packs.
__global__ __launch_bounds__(kKvScanBlock) void kv_scan_totals_kernel(const int32_t* __restrict__ k, int64_t n, int d,
                                                                      int64_t* __restrict__ blocksum, WsHeader* hdr) {
  __shared__ int wsum[kKvScanBlock / 64];
  const int64_t i = (int64_t)blockIdx.x * kKvScanBlock + threadIdx.x;
  if (i == 0) clear_header(hdr);
  int bad = 0;
  const int tot = wave_sum_i(i < n ? seg_len(k[i], d, bad) : 0);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
#pragma unroll
    for (int w = 0; w < kKvScanBlock / 64; ++w) t += wsum[w];
    blocksum[blockIdx.x] = t;
  }
}

// One workgroup: blocksum <- its exclusive prefix sum, four totals per thread and turn.
__global__ __launch_bounds__(1024) void kv_scan_blocks_kernel(int64_t* __restrict__ blocksum, int nblocks) {
  constexpr int PER = 4;
  __shared__ int64_t buf[1024];
  __shared__ int64_t carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (int base = 0; base < nblocks; base += 1024 * PER) {
    const int i = base + threadIdx.x * PER;
    int64_t x[PER], own = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) x[u] = i + u < nblocks ? blocksum[i + u] : 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) own += x[u];
    buf[threadIdx.x] = own;
    __syncthreads();
    for (unsigned o = 1; o < 1024; o <<= 1) {
      const int64_t y = threadIdx.x >= o ? buf[threadIdx.x - o] : 0;
      __syncthreads();
      buf[threadIdx.x] += y;
      __syncthreads();
    }
    const int64_t carry = carry_s;
    int64_t before = carry + buf[threadIdx.x] - own;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (i + u < nblocks) blocksum[i + u] = before;
      before += x[u];
    }
    __syncthreads();
    if (threadIdx.x == 1023) carry_s = carry + buf[1023];
    __syncthreads();
  }
}

// Offsets and copy of the segments, four tokens per wavefront.  A workgroup adds up what lies before its tokens itself.
// kAll (pack_waves below): all the counts before them, L2 reads of at most 128 KB, in one launch; the last workgroup sees
// every count, so it sets the error word and clears the header with one store.  Otherwise (four wavefronts) the totals of the
// blocks before, which a launch of its own has formed (or their prefix sum, when there are so many that `scanned` says so),
// and the tokens before it in its own block.
// A wavefront's four tokens are under way together: one 16-byte chunk per lane of each is requested before the first is
// stored (one token after the other 262144 x 64 took 61.7 us, now 43.6).
constexpr int kPackPer = 4;
template <typename T, int kWaves, bool kAll>
__global__ __launch_bounds__(64 * kWaves) void kv_pack_kernel(const T* __restrict__ xt, const int32_t* __restrict__ k,
                                                              const int64_t* __restrict__ blocksum, int scanned, int64_t n,
                                                              int d, int64_t off_base, int64_t* __restrict__ off,
                                                              T* __restrict__ packed, int64_t capacity, WsHeader* hdr) {
  constexpr int EPC = 16 / (int)sizeof(T);   // elements per 16-byte chunk
  constexpr int TOK = kPackPer * kWaves, NT = 64 * kWaves;
  __shared__ int64_t part[kWaves];
  __shared__ int seg_s[TOK], k_s[TOK], bad_s[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t t0 = (int64_t)blockIdx.x * TOK;
  int bad = 0;
  int64_t before = 0, own;
  if constexpr (kAll) {
    constexpr int U = 8;
    int sum = 0;
    for (int i = threadIdx.x; i < (int)t0; i += NT * U) {
      int kk[U];
#pragma unroll
      for (int u = 0; u < U; ++u) kk[u] = i + u * NT < (int)t0 ? k[i + u * NT] : 0;
#pragma unroll
      for (int u = 0; u < U; ++u) sum += seg_len(kk[u], d, bad);
    }
    before = sum;
    own = t0 + threadIdx.x;
  } else {
    const int64_t blk = t0 / kKvScanBlock;
    if (scanned) {
      if (threadIdx.x == 0) before = blocksum[blk];
    } else {
      for (int64_t i = threadIdx.x; i < blk; i += NT) before += blocksum[i];
    }
    own = blk * kKvScanBlock + threadIdx.x;   // one token of the own block per thread
  }
  if (!kAll || threadIdx.x < TOK) {
    const int own_k = own < n ? k[own] : 0;
    const int own_seg = seg_len(own_k, d, bad);
    if (own < t0) before += own_seg;
    if (own >= t0 && own < t0 + TOK) {
      seg_s[own - t0] = own_seg;
      k_s[own - t0] = min(max(own_k, 0), d);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  const bool wave_bad = __any(bad);
  if (lane == 0) {
    part[wave] = before;
    bad_s[wave] = wave_bad;
  }
  __syncthreads();
  int64_t base = off_base;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) base += part[w];
  if (!kAll && bad && own >= t0 && own < t0 + TOK) atomicOr(&hdr->err, kErrKvCount);
  // every wavefront: the segments' lengths and their exclusive prefix sums, one per lane
  const int lt = lane & (TOK - 1);
  const int seg_l = seg_s[lt], k_l = k_s[lt];
  int excl = seg_l;
#pragma unroll
  for (int o = 1; o < TOK; o <<= 1) {
    const int y = __shfl_up(excl, o, TOK);
    if (lt >= o) excl += y;
  }
  excl -= seg_l;
  if (wave == 0 && lane < TOK && t0 + lane < n) {
    const int64_t o = base + excl;
    off[t0 + lane] = o;
    if (t0 + lane == n - 1) {
      off[n] = o + seg_l;
      if (kAll) {   // the offsets never fall: some segment is out of room if the last one's end is
        int any = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) any |= bad_s[w];
        hdr->err = (any ? kErrKvCount : 0) | (o + seg_l > capacity ? kErrKvCapacity : 0);
        hdr->nv = 0;
      }
    }
    if (!kAll && o + seg_l > capacity) atomicOr(&hdr->err, kErrKvCapacity);
  }
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  u32x4 first[kPackPer];
#pragma unroll
  for (int u = 0; u < kPackPer; ++u) {
    const int ti = u * kWaves + wave;
    const int seg = __builtin_amdgcn_readlane(seg_l, ti);
    // lanes past the segment, and tokens past the last, read what is there and drop it
    first[u] = *reinterpret_cast<const u32x4*>(xt + min(t0 + ti, n - 1) * d + max(min(lane * EPC, seg - EPC), 0));
  }
#pragma unroll
  for (int u = 0; u < kPackPer; ++u) {
    const int ti = u * kWaves + wave;
    const int64_t tok = t0 + ti;
    const int seg = __builtin_amdgcn_readlane(seg_l, ti), kk = __builtin_amdgcn_readlane(k_l, ti);
    const int64_t o = base + __builtin_amdgcn_readlane(excl, ti);
    if (tok >= n || o + seg > capacity) continue;
    for (int c = lane; c * EPC < seg; c += 64) {
      u32x4 v = c == lane ? first[u] : *reinterpret_cast<const u32x4*>(xt + tok * d + c * EPC);
      if ((c + 1) * EPC > kk) {
        T e[EPC];
        __builtin_memcpy(e, &v, 16);
#pragma unroll
        for (int j = 0; j < EPC; ++j)
          if (c * EPC + j >= kk) e[j] = (T)0.0f;
        __builtin_memcpy(&v, e, 16);
      }
      *reinterpret_cast<u32x4*>(packed + o + c * EPC) = v;
    }
  }
}
// Wavefronts of the one-launch form, 0: the counts get a launch of their own.  A workgroup of four, 16 tokens, spreads the copy best but
// adds up 2048 counts a round of loads; one of sixteen, 64 tokens, 8192.  Past two rounds of those the launch is cheaper, but for
// long rows, whose copy covers it.  (8192 components of each of 32768 tokens still add up in 32 bits.)  Store, us, GPU time,
// two launches / sixteen / four:
//   bf16 d 64    n 1500 6.0 / 5.6 / 4.0   4500 6.4 / 5.7 / 5.4   6000 6.5 / 5.7 / 5.4   9000 7.0 / 6.1 / 7.0   16000 7.7 / 6.8 / 9.9
//                16400 7.9 / 7.8   17000 8.2 / 9.4   20000 8.2 / 10.3 / 12.3   32768 10.0 / 12.0 / 21.5
//   bf16 d 1024  n 1000 6.6 / 6.6 / 4.6   6000 7.7 / 7.6 / 6.7   9000 8.5 / 8.1 / 8.5   16000 10.5 / 9.8 / 12.8   16400 10.6 / 10.1
//                17000 10.9 / 12.5   24000 12.6 / 14.3 / 18.5;   d 1536  n 16400 12.4 / 11.4   17000 12.8 / 14.0
//   bf16 d 2048  n 24000 21.8 / 19.8 / 22.7   32768 27.1 / 24.6 / 29.4;   fp32 d 8192  n 700 21.7 / 31.9 / 19.4   6000 49.4 / 47.4 / 46.6
constexpr int64_t kPackFew = 6144, kPackAll = 32768;
constexpr int64_t kPackMost = 2 * 8192 + 64;   // the counts before the last workgroup's tokens are two rounds
constexpr int64_t kPackLongRow = 4096;   // bytes
static_assert(kPackAll * kKvMaxD <= INT32_MAX, "32-bit sums");
constexpr int kPackWaves = 4, kPackAllWaves = 16;
inline int pack_waves(int64_t n, int64_t row_bytes) {
  return n <= kPackFew ? kPackWaves : n <= (row_bytes >= kPackLongRow ? kPackAll : kPackMost) ? kPackAllWaves : 0;
}
static_assert(kKvScanBlock == 64 * kPackWaves && kKvScanBlock % (kPackPer * kPackWaves) == 0 && kPackPer * kPackAllWaves <= 64,
              "one thread per token of a block, one lane per token of a workgroup");

// ---- dense copy of x ------------------------------------------------------------------------

// A wavefront per row, 16 bytes per lane.  Only for rows megabytes apart, of which memory holds few: a launch and little more.
__global__ __launch_bounds__(256) void kv_dense_kernel(const char* __restrict__ x, int64_t pitch, int64_t n, int row_bytes,
                                                       char* __restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= n) return;
  for (int c = (threadIdx.x & 63) * 16; c < row_bytes; c += 64 * 16)
    *reinterpret_cast<uint4*>(out + r * row_bytes + c) = *reinterpret_cast<const uint4*>(x + r * pitch + c);
}

// ---- grouping by contraction length --------------------------------------------------------

// Position of every token in descending order of K-step count.  Block b owns the tokens that block b of
// kv_prepare_kernel counted and derives where its tokens of each bucket start from the counts of all the blocks: the
// longer buckets, then its own bucket in the blocks before it.  The position inside that range comes from an LDS
// counter, so `order` may differ from run to run within a block's share of a bucket; the reconstruction's results do
// not depend on it (a token's output only involves its own row, and extra K-steps of a tile add exact zeros).
// With the counts made by kv_prepare_kernel this replaces seven launches (four fills, counts, starts, scatter; 27 us of
// kernels at 16411 tokens) by one.
// Besides the token, each sorted position gets the byte offset and byte length of the token's segment in the store
// (validated here against the readable extent), so that the reconstruction reads three contiguous arrays instead of chasing
// order -> off, k.  The positions from n to the tile multiple are padded with (-1, out of range, 0).
__global__ __launch_bounds__(256) void kv_scatter_kernel(const int32_t* __restrict__ k,
                                                         const int64_t* __restrict__ off, int64_t n, int64_t ncap,
                                                         int d, int esz, int64_t bytes, int nbuckets,
                                                         const int32_t* __restrict__ hist, int nblocks, int per_block,
                                                         int32_t* __restrict__ order, uint32_t* __restrict__ pos_off,
                                                         int32_t* __restrict__ pos_len, WsHeader* hdr) {
  extern __shared__ int32_t h[];   // [nbuckets] totals, [nbuckets] next free position of this block
  int32_t* const next = h + nbuckets;
  const int blk = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int b = wave; b < nbuckets; b += 4) {
    int tot = 0, mine = 0;
    for (int i = lane; i < nblocks; i += 64) {
      const int c = hist[(int64_t)i * nbuckets + b];
      tot += c;
      mine += i < blk ? c : 0;
    }
    tot = wave_sum_i(tot);
    mine = wave_sum_i(mine);
    if (lane == 0) {
      h[b] = tot;
      next[b] = mine;
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbuckets; b += 256) {
    int longer = 0;
    for (int q = b + 1; q < nbuckets; ++q) longer += h[q];
    next[b] += longer;
  }
  __syncthreads();
  int bad = 0;
  const int64_t t1 = min(n, (int64_t)(blk + 1) * per_block);
  for (int64_t i = (int64_t)blk * per_block + threadIdx.x; i < t1; i += 256) {
    const int kk = k[i];
    const int64_t o = off[i];
    const int pos = atomicAdd(&next[bucket_of(kk, d, esz)], 1);
    int clamped = 0;
    const int seg = seg_len(kk, d, clamped);
    const bool outside = o < 0 || (o & (DYNAKV_GRANULE - 1)) || (o + seg) * esz > bytes;
    if (outside) bad = 1;
    order[pos] = (int32_t)i;
    pos_len[pos] = seg * esz;
    pos_off[pos] = outside ? 0x80000000u : (uint32_t)(o * esz);   // out of range: every load of the row gives zeros
  }
  if (bad) atomicOr(&hdr->err, kErrKvCapacity);
  if (blk == 0) {
    for (int64_t p = n + threadIdx.x; p < ncap; p += 256) {
      order[p] = -1;
      pos_len[p] = 0;
      pos_off[p] = 0x80000000u;
    }
  }
}

// Where kv_group_fits, one launch instead of two: a workgroup sorts kKvGroup tokens by itself, in LDS.  The tiles of a group
// are then a little less even than those of all the tokens (16 tiles of 128 tokens each, about half a K-step of 7.5 more), which costs
// less than the counts' launch did.  Rank r tiles of all groups come before the rank r + 1 tiles, so that the long ones still start
// first; only the last group can have fewer tiles than the others.
__global__ __launch_bounds__(1024) void kv_group_kernel(const int32_t* __restrict__ k, const int64_t* __restrict__ off,
                                                        int64_t n, int d, int esz, int64_t bytes, int nbuckets, int edge,
                                                        int32_t* __restrict__ order, uint32_t* __restrict__ pos_off,
                                                        int32_t* __restrict__ pos_len, int32_t* __restrict__ outside_out) {
  constexpr int PER = kKvGroup / 1024;
  extern __shared__ int32_t h[];   // [nbuckets] tokens, [nbuckets] first rank
  int32_t* const start = h + nbuckets;
  const int groups = gridDim.x, g = blockIdx.x;
  const int g0 = g * kKvGroup, gn = min((int)n - g0, kKvGroup);
  const int last_tiles = ((int)n - (groups - 1) * kKvGroup + edge - 1) / edge;
  for (int i = threadIdx.x; i < nbuckets; i += 1024) h[i] = 0;
  int kk[PER];
  int64_t o[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = u * 1024 + threadIdx.x;
    kk[u] = i < gn ? k[g0 + i] : 0;
    o[u] = i < gn ? off[g0 + i] : 0;
  }
  __syncthreads();
  int rank[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u)
    rank[u] = u * 1024 + (int)threadIdx.x < gn ? atomicAdd(&h[bucket_of(kk[u], d, esz)], 1) : 0;
  __syncthreads();
  for (int b = threadIdx.x; b < nbuckets; b += 1024) {
    int longer = 0;
    for (int q = b + 1; q < nbuckets; ++q) longer += h[q];
    start[b] = longer;
  }
  __syncthreads();
  auto position = [&](int p) {
    const int r = p / edge;
    const int tile = r < last_tiles ? r * groups + g : last_tiles * groups + (r - last_tiles) * (groups - 1) + g;
    return tile * edge + p % edge;
  };
  int bad = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = u * 1024 + threadIdx.x;
    if (i >= gn) continue;
    int clamped = 0;
    const int seg = seg_len(kk[u], d, clamped);
    const bool outside = o[u] < 0 || (o[u] & (DYNAKV_GRANULE - 1)) || (o[u] + seg) * esz > bytes;
    if (outside) bad = 1;
    const int pos = position(start[bucket_of(kk[u], d, esz)] + rank[u]);
    order[pos] = g0 + i;
    pos_len[pos] = seg * esz;
    pos_off[pos] = outside ? 0x80000000u : (uint32_t)(o[u] * esz);   // out of range: every load of the row gives zeros
  }
  // the rest of the last group's last tile
  for (int p = gn + threadIdx.x; p < (gn + edge - 1) / edge * edge; p += 1024) {
    const int pos = position(p);
    order[pos] = -1;
    pos_len[pos] = 0;
    pos_off[pos] = 0x80000000u;
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) outside_out[g] = bad;
}

// ---- retain rate ----------------------------------------------------------------------------

// Sums of k and of m over tokens [t0, t0 + tn), valid in thread 0; a workgroup of NT threads.
template <int NT>
__device__ inline void retain_sums(const int32_t* __restrict__ k, const float* __restrict__ m, int64_t t0, int64_t tn, int d,
                                   double& ks, double& ms) {
  __shared__ double sk[NT / 64], sm[NT / 64];
  ks = 0.0;
  if (k)
    for (int64_t i = threadIdx.x; i < tn; i += NT) ks += min(max(k[t0 + i], 0), d);
  ms = 0.0;
  if (m) {
    const int64_t cnt4 = tn * d / 4;
    const float4* p = reinterpret_cast<const float4*>(m + t0 * d);
    for (int64_t i = threadIdx.x; i < cnt4; i += 4 * NT) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = i + NT * u < cnt4 ? p[i + NT * u] : make_float4(0.f, 0.f, 0.f, 0.f);
      float t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = (v[u].x + v[u].y) + (v[u].z + v[u].w);
      ms += (double)((t[0] + t[1]) + (t[2] + t[3]));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ks += __shfl_xor(ks, o);
    ms += __shfl_xor(ms, o);
  }
  if ((threadIdx.x & 63) == 0) {
    sk[threadIdx.x >> 6] = ks;
    sm[threadIdx.x >> 6] = ms;
  }
  __syncthreads();
  ks = ms = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < NT / 64; ++w) {
      ks += sk[w];
      ms += sm[w];
    }
}
__device__ inline void retain_out(double ks, double ms, bool have_k, bool have_m, double nd, float alpha,
                                  float* __restrict__ out) {
  const double rh = have_k ? ks / nd : 0.0, rs = have_m ? ms / nd : 0.0;
  out[0] = (float)rh;
  out[1] = (float)rs;
  out[2] = (float)(alpha * rs * rs);
}

// red[2*b] = sum of k over the block's tokens, red[2*b+1] = sum of m over their rows.  The tokens are cut evenly over
// the blocks.  Bound by the one read of m: as many blocks as the chip holds at once (kKvRetainBlocks), each thread with
// four loads in flight.  (One block per 256 tokens gave 16 blocks for 4096 tokens and 66 us, now 5.5.)
__global__ __launch_bounds__(256) void kv_retain_partial_kernel(const int32_t* __restrict__ k,
                                                                const float* __restrict__ m, int64_t n, int d,
                                                                double* __restrict__ red, WsHeader* hdr) {
  if (blockIdx.x == 0 && threadIdx.x == 0) clear_header(hdr);
  const int64_t t0 = n * blockIdx.x / gridDim.x;
  double ks, ms;
  retain_sums<256>(k, m, t0, n * (blockIdx.x + 1) / gridDim.x - t0, d, ks, ms);
  if (threadIdx.x == 0) {
    red[2 * blockIdx.x] = ks;
    red[2 * blockIdx.x + 1] = ms;
  }
}

// Few values (kRetainFew): one workgroup and one launch.
__global__ __launch_bounds__(1024) void kv_retain_few_kernel(const int32_t* __restrict__ k, const float* __restrict__ m,
                                                             int64_t n, int d, float alpha, float* __restrict__ out,
                                                             WsHeader* hdr) {
  double ks, ms;
  retain_sums<1024>(k, m, 0, n, d, ks, ms);
  if (threadIdx.x == 0) {
    clear_header(hdr);
    retain_out(ks, ms, k != nullptr, m != nullptr, (double)n * d, alpha, out);
  }
}

// One block.  Eight pairs in flight per thread, then a tree over the threads.
__global__ __launch_bounds__(256) void kv_retain_final_kernel(const double* __restrict__ red, int nblocks,
                                                              int64_t n, int d, float alpha, int have_k,
                                                              int have_m, float* __restrict__ out) {
  __shared__ double sk[4], sm[4];
  double a = 0.0, b = 0.0;
#pragma unroll
  for (int u = 0; u < kKvRetainBlocks / 256; ++u) {
    const int i = threadIdx.x + 256 * u;
    if (i < nblocks) {
      a += red[2 * i];
      b += red[2 * i + 1];
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o);
    b += __shfl_xor(b, o);
  }
  if ((threadIdx.x & 63) == 0) {
    sk[threadIdx.x >> 6] = a;
    sm[threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    retain_out((sk[0] + sk[1]) + (sk[2] + sk[3]), (sm[0] + sm[1]) + (sm[2] + sm[3]), have_k, have_m, (double)n * d, alpha,
               out);
}

__global__ __launch_bounds__(256) void kv_retain_grad_kernel(const float* __restrict__ out, float alpha,
                                                             int64_t count4, double nd, float* __restrict__ g) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count4) return;
  const float v = (float)(2.0 * alpha * (double)out[1] / nd);
  reinterpret_cast<float4*>(g)[i] = make_float4(v, v, v, v);
}

}  // namespace

template <typename T>
static void launch_mask_t(const float* logits, const float* b, const void* xt, int64_t n, int d, float tau,
                          bool literal, int32_t* k, float* m, void* xhat, hipStream_t s) {
  const dim3 grid((unsigned)((n + 3) / 4));
  const T* x = static_cast<const T*>(xt);
  T* xh = static_cast<T*>(xhat);
  const int lit = literal ? 1 : 0;
  const int ng = (d + 255) / 256;
#define KV_MASK(NG) hipLaunchKernelGGL((kv_mask_kernel<T, NG>), grid, dim3(256), 0, s, logits, b, x, n, d, tau, lit, k, m, xh)
  switch (ng) {
    case 1: KV_MASK(1); break;
    case 2: KV_MASK(2); break;
    case 3: KV_MASK(3); break;
    case 4: KV_MASK(4); break;
    case 5: case 6: KV_MASK(6); break;
    case 7: case 8: KV_MASK(8); break;
    default: KV_MASK(0); break;
  }
#undef KV_MASK
}

hipError_t launch_kv_mask(int dtype, const float* logits, const float* b, const void* xt, int64_t n, int d,
                          float tau, bool literal, int32_t* k, float* m, void* xhat, hipStream_t s) {
  if (dtype == LMHEAD_BF16)
    launch_mask_t<__bf16>(logits, b, xt, n, d, tau, literal, k, m, xhat, s);
  else
    launch_mask_t<float>(logits, b, xt, n, d, tau, literal, k, m, xhat, s);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_mask_bwd_t(const float* logits, const float* b, const void* xt, const void* g_xhat,
                                    const float* g_m, float g_m_const, int64_t n, int d, bool literal, void* gl,
                                    void* a_out, float* dbpart, int nblk, int32_t* clear, int nclear, hipStream_t s) {
  const dim3 grid((unsigned)nblk);
  const size_t lds = (size_t)4 * d * sizeof(float);
  const T* x = static_cast<const T*>(xt);
  const T* gx = static_cast<const T*>(g_xhat);
  T* g1 = static_cast<T*>(gl);
  T* a1 = static_cast<T*>(a_out);
  const int lit = literal ? 1 : 0;
  const int ng = (d + 255) / 256;
#define KV_MASK_BWD(NG)                                                                                          \
  do {                                                                                                           \
    hipError_t e = allow_lds<kv_mask_bwd_kernel<T, NG>>((int)lds);                                               \
    if (e != hipSuccess) return e;                                                                               \
    hipLaunchKernelGGL((kv_mask_bwd_kernel<T, NG>), grid, dim3(256), lds, s, logits, b, x, gx, g_m, g_m_const, n, \
                       d, lit, g1, a1, dbpart, clear, nclear);                                                   \
  } while (0)
  switch (ng) {
    case 1: KV_MASK_BWD(1); break;
    case 2: KV_MASK_BWD(2); break;
    case 3: KV_MASK_BWD(3); break;
    case 4: KV_MASK_BWD(4); break;
    case 5: case 6: KV_MASK_BWD(6); break;
    case 7: case 8: KV_MASK_BWD(8); break;
    default: KV_MASK_BWD(0); break;
  }
#undef KV_MASK_BWD
  return hipGetLastError();
}

hipError_t launch_kv_mask_bwd(int dtype, const float* logits, const float* b, const void* xt, const void* g_xhat,
                              const float* g_m, float g_m_const, int64_t n, int d, bool literal, void* gl,
                              void* a_out, float* dbpart, int nblk, int32_t* clear, int nclear, hipStream_t s) {
  if (dtype == LMHEAD_BF16)
    return launch_mask_bwd_t<__bf16>(logits, b, xt, g_xhat, g_m, g_m_const, n, d, literal, gl, a_out, dbpart, nblk, clear, nclear, s);
  return launch_mask_bwd_t<float>(logits, b, xt, g_xhat, g_m, g_m_const, n, d, literal, gl, a_out, dbpart, nblk, clear, nclear, s);
}

hipError_t launch_kv_sums(const KvSums& a, hipStream_t s) {
  constexpr int64_t NT = 64 * kSumWaves;
  const bool by_columns = a.d <= kSumByColumns;
  const int64_t columns = a.slices > 1 ? 2 * (int64_t)a.d * a.d : 0, per_block = by_columns ? 64 : 4 * NT;   // of both gradients
  hipLaunchKernelGGL(kv_sum_kernel, dim3((unsigned)(a.d / 64 + (columns + per_block - 1) / per_block)), dim3((unsigned)NT), 0, s, a,
                     by_columns ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_kv_prepare(int esz, const KvPrepareArgs& a, hipStream_t s) {
  const int64_t blocks = a.count.blocks + (a.njobs > 0 ? (int64_t)a.njobs * (a.job[0].d / 64) * (a.job[0].d / 64) : 0);
  hipLaunchKernelGGL(kv_prepare_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a, esz);
  return hipGetLastError();
}

hipError_t launch_kv_store(int dtype, const void* xt, const int32_t* k, int64_t n, int d, int64_t off_base,
                           int64_t* off, void* packed, int64_t capacity, int64_t* blocksum, WsHeader* hdr,
                           hipStream_t s) {
  const int64_t nblocks = (n + kKvScanBlock - 1) / kKvScanBlock;
  // Up to kScanFrom blocks every packing workgroup adds up the totals before it by itself (4 loads per thread at
  // the most); beyond, that would grow with the square of n and one workgroup forms the prefix sums first (whole call,
  // tokens of 64 components: 524288 86.2 us without it, 79.4 with it).
  constexpr int64_t kScanFrom = 1024;
  const int scanned = nblocks > kScanFrom ? 1 : 0;
  const int all = pack_waves(n, (int64_t)d * (dtype == LMHEAD_BF16 ? 2 : 4));
  if (!all)
    hipLaunchKernelGGL(kv_scan_totals_kernel, dim3((unsigned)nblocks), dim3(kKvScanBlock), 0, s, k, n, d, blocksum, hdr);
  if (scanned) hipLaunchKernelGGL(kv_scan_blocks_kernel, dim3(1), dim3(1024), 0, s, blocksum, (int)nblocks);
  const int waves = all ? all : kPackWaves;
  const dim3 grid((unsigned)((n + kPackPer * waves - 1) / (kPackPer * waves))), block(64 * waves);
  auto launch = [&](auto kernel, auto* x, auto* out) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, x, k, blocksum, scanned, n, d, off_base, off, out, capacity, hdr);
  };
  auto typed = [&](auto* x, auto* out) {
    using T = std::remove_reference_t<decltype(*out)>;
    if (all == kPackWaves)
      launch(kv_pack_kernel<T, kPackWaves, true>, x, out);
    else if (all)
      launch(kv_pack_kernel<T, kPackAllWaves, true>, x, out);
    else
      launch(kv_pack_kernel<T, kPackWaves, false>, x, out);
  };
  if (dtype == LMHEAD_BF16)
    typed(static_cast<const __bf16*>(xt), static_cast<__bf16*>(packed));
  else
    typed(static_cast<const float*>(xt), static_cast<float*>(packed));
  return hipGetLastError();
}

hipError_t launch_kv_dense(const void* x, int64_t pitch, int64_t n, int row_bytes, void* out, hipStream_t s) {
  hipLaunchKernelGGL(kv_dense_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, static_cast<const char*>(x), pitch, n,
                     row_bytes, static_cast<char*>(out));
  return hipGetLastError();
}

hipError_t launch_kv_order(int dtype, const KvCount& c, const int64_t* off, int64_t bytes, int64_t ncap, int32_t* order,
                           uint32_t* pos_off, int32_t* pos_len, WsHeader* hdr, hipStream_t s) {
  const int esz = dtype == LMHEAD_BF16 ? 2 : 4;
  hipLaunchKernelGGL(kv_scatter_kernel, dim3((unsigned)c.blocks), dim3(256), 2 * c.nbuckets * sizeof(int32_t), s, c.k,
                     off, c.n, ncap, c.d, esz, bytes, c.nbuckets, c.hist, c.blocks, c.per_block, order, pos_off, pos_len,
                     hdr);
  return hipGetLastError();
}

hipError_t launch_kv_group(int dtype, const int32_t* k, const int64_t* off, int64_t n, int d, int64_t bytes, int nbuckets, int edge,
                           int32_t* order, uint32_t* pos_off, int32_t* pos_len, int32_t* outside, hipStream_t s) {
  const int esz = dtype == LMHEAD_BF16 ? 2 : 4;
  hipLaunchKernelGGL(kv_group_kernel, dim3((unsigned)((n + kKvGroup - 1) / kKvGroup)), dim3(1024),
                     2 * nbuckets * sizeof(int32_t), s, k, off, n, d, esz, bytes, nbuckets, edge, order, pos_off, pos_len, outside);
  return hipGetLastError();
}

hipError_t launch_kv_retain(const int32_t* k, const float* m, int64_t n, int d, float alpha, float* out,
                            float* g_m, double* red, WsHeader* hdr, hipStream_t s) {
  // Up to here one workgroup reads everything sooner than two launches do.  GPU time, us, two launches / one: 1024 values 4.2 / 2.8,
  // 32768 4.8 / 3.4, 65536 4.9 / 4.0, 96000 7.0 / 5.0 (1500 x 64), 102400 4.7 / 5.2 (100 x 1024), 131584 4.8 / 5.8, 204800 4.8 / 8.0.
  // (A caller that enqueues nothing else waits for the host instead, 11 us for two launches, 8 for one.)
  constexpr int64_t kRetainFew = 98304;
  if (n * d <= kRetainFew) {
    hipLaunchKernelGGL(kv_retain_few_kernel, dim3(1), dim3(1024), 0, s, k, m, n, d, alpha, out, hdr);
  } else {
    const int nblocks = (int)(n < kKvRetainBlocks ? n : kKvRetainBlocks);
    hipLaunchKernelGGL(kv_retain_partial_kernel, dim3(nblocks), dim3(256), 0, s, k, m, n, d, red, hdr);
    hipLaunchKernelGGL(kv_retain_final_kernel, dim3(1), dim3(256), 0, s, red, nblocks, n, d, alpha, k ? 1 : 0,
                       m ? 1 : 0, out);
  }
  if (g_m) {
    const int64_t count4 = n * d / 4;
    hipLaunchKernelGGL(kv_retain_grad_kernel, dim3((unsigned)((count4 + 255) / 256)), dim3(256), 0, s, out, alpha,
                       count4, (double)n * d, g_m);
  }
  return hipGetLastError();
}

}  // namespace lmhead
