// The truncation mask of one token by one wavefront (Eqs. 5-8), used by the mask's own kernel and by the few-token product whose last
// workgroup applies it.
#pragma once

#include "dynakv_common.h"

namespace lmhead {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ inline int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

template <typename T>
struct Store4;
template <>
struct Store4<float> {
  __device__ static inline void load(const float* p, float (&v)[4]) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
  __device__ static inline void store(float* p, const float (&v)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  }
};
template <>
struct Store4<__bf16> {
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
  __device__ static inline void load(const __bf16* p, float (&v)[4]) {
    const bf16x4_t t = *reinterpret_cast<const bf16x4_t*>(p);
    v[0] = (float)t.x; v[1] = (float)t.y; v[2] = (float)t.z; v[3] = (float)t.w;
  }
  __device__ static inline void store(__bf16* p, const float (&v)[4]) {
    const bf16x4_t t = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    *reinterpret_cast<bf16x4_t*>(p) = t;
  }
};

// Mask position i belongs to gate column j(i) = i (reverse cumulative
// sum) or j(i) = d-1-i (Eq. 6 as printed: Flip(cumsum(p))_i = sum_{i' >= i} p_{d-1-i'}), so both
// readings are the same suffix sum over positions.  Positions are walked in groups of 256 (four
// per lane, contiguous), last group first, carrying the running suffix.
// NG > 0: the row has NG groups (d <= 256 NG) and is held in registers: one pass over memory.
// NG == 0: any d; the row of logits is read three times (max, sum, suffix), the second and third
// time from L1/L2.
// row4(j): the logits of columns j to j + 3.  Returns the number of positions above tau, in every lane.
template <typename T, int NG, typename Load>
__device__ inline int mask_token(Load&& row4, const float* __restrict__ bias, const T* __restrict__ xt, int64_t tok, int d, float tau,
                                 int literal, float* __restrict__ m_out, T* __restrict__ xhat) {
  const int lane = threadIdx.x & 63;
  const int ngroups = NG > 0 ? NG : (d + 255) / 256;

  // logits (+ bias) of the four positions that start at i0, in position order
  auto load4 = [&](int i0, float (&v)[4]) {
    const int j0 = literal ? d - 4 - i0 : i0;   // literal: columns j0 .. j0+3 are positions i0+3 .. i0
    const float4 a = row4(j0);
    const float4 b = *reinterpret_cast<const float4*>(bias + j0);
    if (!literal) {
      v[0] = a.x + b.x; v[1] = a.y + b.y; v[2] = a.z + b.z; v[3] = a.w + b.w;
    } else {
      v[0] = a.w + b.w; v[1] = a.z + b.z; v[2] = a.y + b.y; v[3] = a.x + b.x;
    }
  };

  constexpr int NR = NG > 0 ? NG : 1;
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
        row[g][e] = __builtin_amdgcn_exp2f((row[g][e] - mx) * kLog2e);   // exp(-inf) = 0 beyond d
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

  float carry = 0.f;   // sum of exp over all positions after the current group
  int count = 0;
  // one group: s[] = the lane's four exponentials in position order
  auto group = [&](int g, float (&s)[4]) {
    const int i0 = g * 256 + lane * 4;
    const bool on = i0 < d;
    s[2] += s[3];
    s[1] += s[2];
    s[0] += s[1];
    // inclusive suffix sum of the lanes' totals (this lane and the lanes above it)
    float incl = s[0];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const float y = __shfl_down(incl, o);
      if (lane + o < 64) incl += y;
    }
    const float above = carry + (incl - s[0]);
    carry += __shfl(incl, 0);
    if (on) {
      float mk[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        mk[e] = (above + s[e]) * inv;
        count += mk[e] > tau ? 1 : 0;
      }
      if (m_out) Store4<float>::store(m_out + tok * d + i0, mk);
      if (xhat) {
        float xv[4];
        Store4<T>::load(xt + tok * d + i0, xv);
#pragma unroll
        for (int e = 0; e < 4; ++e) xv[e] *= mk[e];
        Store4<T>::store(xhat + tok * d + i0, xv);
      }
    }
  };
  if constexpr (NG > 0) {
#pragma unroll
    for (int g = NG - 1; g >= 0; --g) group(g, row[g]);
  } else {
    for (int g = ngroups - 1; g >= 0; --g) {
      const int i0 = g * 256 + lane * 4;
      float s[4] = {0.f, 0.f, 0.f, 0.f};
      if (i0 < d) {
        float v[4];
        load4(i0, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_exp2f((v[e] - mx) * kLog2e);
      }
      group(g, s);
    }
  }
  return wave_sum_i(count);
}

}  // namespace

}  // namespace lmhead
