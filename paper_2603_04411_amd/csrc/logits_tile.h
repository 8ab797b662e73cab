// What the forward does with a finished tile of logits: the target's logit and the softmax statistics of each token.
#pragma once

#include <type_traits>

#include "common.h"
#include "gemm_core.h"

namespace lmhead {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegInf = -__builtin_huge_valf(), kLowest = -__FLT_MAX__;

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Merge (m2, s2, t2) into (m, s, t): statistics of a union of disjoint logit sets.
__device__ inline void merge_stats(float& m, float& s, float& t, float m2, float s2, float t2) {
  const float mn = fmaxf(m, m2);
  const float ms = (mn == kNegInf) ? 0.f : mn;
  const float a = fast_exp2((m - ms) * kLog2e);
  const float b = fast_exp2((m2 - ms) * kLog2e);
  s = s * a + s2 * b;
  t = t * a + t2 * b;
  m = mn;
}

// Target-logit capture: only where some lane's target (tkj: its token columns' ids) falls inside this tile, rows m0 to m_end.
template <typename G>
__device__ inline void capture_target(const FwdArgs& a, typename G::Acc& acc, const int (&tkj)[G::TN], int m0, int m_end, int64_t n0,
                                      float* __restrict__ zy, int32_t* __restrict__ gid) {
  int relj[G::TN];
  bool hit = false;
#pragma unroll
  for (int j = 0; j < G::TN; ++j) {
    const int tk = tkj[j];
    const bool in = (tk >= m0) & (tk < m_end);
    hit |= in;
    relj[j] = m_end - m0 == G::BM || in ? tk - m0 - G::m_base() : -1;   // compared with compile-time constants
  }
  if (__any(hit)) {
#pragma unroll
    for (int j = 0; j < G::TN; ++j) {
      float zsel = 0.f;
      bool found = false;
#pragma unroll
      for (int i = 0; i < G::TM; ++i)
#pragma unroll
        for (int v = 0; v < G::VB; ++v) {
          const bool eq = relj[j] == G::m_const(i, v);
          zsel = eq ? acc[i][j][v] : zsel;
          found |= eq;
        }
      if (found) {
        zy[n0 + G::n_of(j)] = zsel * a.zscale;
        // vocabulary column of the accumulator element just selected (the compare above held for it)
        gid[n0 + G::n_of(j)] = m0 + G::m_base() + relj[j];
      }
    }
  }
}

// Softmax statistics of this lane's token columns, to which a tile's are added.
template <typename G>
struct TileStats {
  float m[G::TN], s[G::TN], t[G::TN];
  __device__ inline void clear() {
#pragma unroll
    for (int j = 0; j < G::TN; ++j) {
      m[j] = kNegInf;
      s[j] = 0.f;
      t[j] = 0.f;
    }
  }
  // Inside the lane, 16 values of one token column at a time (one 32x32 block or four 16x16 blocks); the scheduling
  // barrier after each group keeps the accumulator reads of later groups from being hoisted, so only 16 values are live
  // in VGPRs at a time.  vlim: rows with m_const >= vlim do not count (whole: there are none).  want_t: the third sum is needed.
  // A logit of -inf (a masked row of W) does not count either, in any of the three: its exponential is 0.
  __device__ inline void add(typename G::Acc& acc, float zscale, int vlim, bool whole, bool want_t) {
    // logit = accumulator * zscale (zscale = 1 unless the operands are scaled 8-bit copies); the factor
    // is folded into the constants of the group instead of being applied per element
    const float kz = kLog2e * zscale;
    constexpr int BPC = 16 / G::VB < G::TM ? 16 / G::VB : G::TM;   // blocks per group
    constexpr int GV = BPC * G::VB;            // values per group: 16 (8 in the 64 wide bf16 tile)
    static_assert(G::TM % BPC == 0 && GV % 2 == 0, "whole groups");
    auto group_stats = [&](auto full_tag, auto ent_tag, int ic, int j, float& m_run, float& s_run, float& t_run) {
      constexpr bool kFull = decltype(full_tag)::value;
      constexpr bool kEnt = decltype(ent_tag)::value;   // the third accumulator (sum exp * z) feeds the entropy only
      float z[GV];
#pragma unroll
      for (int b = 0; b < BPC; ++b)
#pragma unroll
        for (int v = 0; v < G::VB; ++v)
          z[b * G::VB + v] = kFull || G::m_const(ic * BPC + b, v) < vlim ? acc[ic * BPC + b][j][v] : kNegInf;
      float tmax = fmaxf(z[0], z[1]);
#pragma unroll
      for (int v = 2; v < GV; v += 2) tmax = fmaxf(tmax, fmaxf(z[v], z[v + 1]));
      const float mn = fmaxf(m_run, tmax * zscale);
      const float ms = (mn == kNegInf) ? 0.f : mn;
      const float sc = fast_exp2((m_run - ms) * kLog2e);
      const float bias = -ms * kLog2e;
      float ss = 0.f, ts = 0.f;
#pragma unroll
      for (int v = 0; v < GV; ++v) {
        const float e = fast_exp2(fmaf(z[v], kz, bias));   // exp2(-inf) = 0 on padding rows
        ss += e;
        if constexpr (kEnt) ts = fmaf(e, fmaxf(z[v], kLowest), ts);   // 0 * -inf would be NaN
      }
      s_run = fmaf(s_run, sc, ss);
      if constexpr (kEnt) t_run = fmaf(t_run, sc, ts * zscale);
      m_run = mn;
      __builtin_amdgcn_sched_barrier(0);
    };
    auto all_groups = [&](auto full_tag, auto ent_tag) {
#pragma unroll
      for (int j = 0; j < G::TN; ++j)
#pragma unroll
        for (int ic = 0; ic < G::TM / BPC; ++ic) group_stats(full_tag, ent_tag, ic, j, m[j], s[j], t[j]);
    };
    if (whole) {
      if (want_t) all_groups(std::true_type{}, std::true_type{}); else all_groups(std::true_type{}, std::false_type{});
    } else {
      if (want_t) all_groups(std::false_type{}, std::true_type{}); else all_groups(std::false_type{}, std::false_type{});
    }
  }
  // The lane groups of a block (same token, other vocabulary rows), into LDS (`red`: [WGM][BN][3]).
  __device__ inline void to_lds(float* red) {
#pragma unroll
    for (int j = 0; j < G::TN; ++j) {
#pragma unroll
      for (int o = 32; o >= G::NB; o >>= 1) {
        const float m2 = __shfl_xor(m[j], o);
        const float s2 = __shfl_xor(s[j], o);
        const float t2 = __shfl_xor(t[j], o);
        merge_stats(m[j], s[j], t[j], m2, s2, t2);
      }
      if (G::lane() < G::NB) {
        float* q = red + ((size_t)G::wave_m() * G::BN + G::n_of(j)) * 3;
        q[0] = m[j];
        q[1] = s[j];
        q[2] = t[j];
      }
    }
  }
  // Behind a barrier, the WGM waves of a token, into plane `tile` of part.
  __device__ inline void store(const FwdArgs& a, const float* red, float* __restrict__ part, int tile, int64_t n0, bool want_t) {
    lds_barrier();
    for (int n = threadIdx.x; n < G::BN; n += G::NT) {
      float mw = red[n * 3], sw = red[n * 3 + 1], tw = red[n * 3 + 2];
#pragma unroll
      for (int w = 1; w < G::WGM; ++w) {
        const float* q = red + ((size_t)w * G::BN + n) * 3;
        merge_stats(mw, sw, tw, q[0], q[1], q[2]);
      }
      const size_t base = (size_t)tile * a.Ncap + n0 + n;
      const size_t plane = (size_t)a.ntiles * a.Ncap;
      part[base] = mw;
      part[plane + base] = sw;
      if (want_t) part[2 * plane + base] = tw;
    }
  }
};

}  // namespace

}  // namespace lmhead
