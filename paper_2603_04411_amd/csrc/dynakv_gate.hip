// The gate over many tokens in one kernel (Eqs. 1, 5, 6, 8): x~ = x U, logits x~ W + b, softmax, cumulative mask and the
// count of components above the threshold, without the logits ever leaving the registers.  For callers that do not
// ask for the soft mask or x^ (prefill, decoding); training takes the separate kernels.
//
// A workgroup owns TOK = 16 TJ tokens and ALL d output columns of both products, so that a token's softmax
// never crosses workgroups: eight wavefronts, each d / 8 columns x TOK tokens of 16x16 MFMA blocks (128 accumulator
// registers; two on a SIMD, which cover each other's waits).  The token rows (TOK x d bf16, 128 KB) sit in LDS for the whole
// product and are read by all wavefronts; the parameter matrices stream from L2 straight into registers, each value into the one wavefront that
// needs it, in fragments of 1 KB that kv_prepare_kernel has laid out in the order they are consumed (a full-line
// load per instruction, no LDS, no barrier in the main loop).  A fragment register is reloaded right behind
// its last use, two K sub-steps ahead (about 2000 cycles).
//
// What bounds it: the parameter stream.  Every 64 tokens read 2 d^2 x 2 bytes (4 MB at d = 1024) through a compute unit's
// 64 bytes per clock, which just matches the matrix cores' pace; 256 x 256 tiles need half of that but pay a pipeline
// fill and an epilogue per 16 K-steps, one write and one read of the fp32 logits and one read of x~ (3.2 GB at
// 262144 x 1024).  Measured there: 1334 us with the separate kernels, 1038 with four wavefronts, 981 now (d = 512: 309, now 296;
// 16384 x 1024: 78, now 75).  Of a round's 60 us (sixteen rounds) the matrix pipe is busy for 34, the softmax takes 8.  Beginning the
// contractions at another sub-step in each workgroup, so that they do not read the same parameters at a time: the second
// alone nothing (979; d = 512: 300), both up to 4 %, but a token's sums would depend on its place in the call.
//
// Column order: accumulator element v of block i in lane group q of wavefront w is POSITION (d/8) w + (d/32) q + 4 i + v of
// the mask, i.e. a lane holds d / 32 consecutive positions of one token per token block, and the cumulative sum is a
// loop inside the lane plus an exchange of 32 partial sums per token.  (Position p is gate column p, or d - 1 - p for
// Eq. 6 as printed; the fragment layout of W and the bias follow that order.)
#include "dynakv_common.h"
#include "gemm_core.h"

#include <type_traits>

namespace lmhead {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

template <int NI_, int TJ_>
struct Gate {
  static constexpr int NI = NI_, TJ = TJ_, NW = kKvGateWaves;   // 16-row blocks of columns per wavefront, 16-token blocks, wavefronts
  static constexpr int D = 16 * NW * NI;
  static constexpr int TOK = 16 * TJ;
  static constexpr int S = D / 32;              // K sub-steps of one MFMA each
  static constexpr int ROW = D * 2;             // bytes of a token row
  static constexpr int PITCH = ROW + 16;        // in LDS: 16 rows' chunks fall on different banks
  static constexpr int X_BYTES = TOK * PITCH;
  static constexpr int BIAS_OFF = X_BYTES, RED_OFF = BIAS_OFF + D * 4;
  static constexpr int LDS_BYTES = RED_OFF + 3 * NW * TOK * 4;
  static constexpr int STEP = NI * 1024;        // bytes of one wavefront's fragments per sub-step
  static constexpr int PIECES = TOK / NW * (ROW / 1024);   // 1 KB pieces of token rows per wavefront
  static_assert((ROW == 1024 || ROW == 2048) && (PIECES % S == 0 || S % PIECES == 0) && S % 2 == 0 && S >= 6 && LDS_BYTES <= 160 * 1024, "tile shape");
};

template <typename G>
__global__ __launch_bounds__(64 * kKvGateWaves) void kv_gate_kernel(KvGateArgs a) {
  typedef __attribute__((address_space(3))) void* lptr_t;
  constexpr int NI = G::NI, TJ = G::TJ, NW = G::NW, S = G::S;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float* const bias_s = reinterpret_cast<float*>(smem + G::BIAS_OFF);
  float* const red = reinterpret_cast<float*>(smem + G::RED_OFF);   // [3][NW][TOK]
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // The lane number, opaque to the optimiser: every phase derives its addresses from it anew.  (Hoisted out of the
  // tile loop they were 25 registers too many, and each reload from scratch memory in the loop a wait for
  // everything in flight.)
  auto lane_id = []() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    return l;
  };

  // The two streams of fragments, x and x~ as buffers.  A row past the last token lies outside them by its offset
  // alone (less than 2^32: kv_gate_fits): its loads give zeros, its stores are dropped.
  auto rsrc = [](const void* p, int64_t bytes) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), 0,
                                             (int)__builtin_amdgcn_readfirstlane((uint32_t)bytes), 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t rU = rsrc(a.Ufrag, (int64_t)G::D * G::D * 2), rW = rsrc(a.Wfrag, (int64_t)G::D * G::D * 2);
  const __amdgpu_buffer_rsrc_t rX = rsrc(a.x, ((a.n - 1) * a.ldx + G::D) * 2), rXt = rsrc(a.xt, a.n * G::D * 2);
  const int woff = w * S * G::STEP;   // this wavefront's part of a stream

  for (int c = threadIdx.x; c < G::D; c += 64 * NW) bias_s[c] = a.bias[a.literal ? G::D - 1 - c : c];

  // 1 KB piece p of this wavefront's token rows: tile row and byte within it
  auto piece_row = [&](int p) { return w * (G::TOK / NW) + p / (G::ROW / 1024); };
  auto piece_col = [&](int p) { return p % (G::ROW / 1024) * 1024; };
  auto load_x = [&](int64_t t0) {
    const uint32_t pitch = (uint32_t)(a.ldx * 2);
    uint32_t vo = lane_id() * 16 + (uint32_t)(t0 + piece_row(0)) * pitch;
#pragma unroll 4
    for (int p = 0; p < G::PIECES; p += G::ROW / 1024) {
      char* const dst = smem + piece_row(p) * G::PITCH;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rX, (lptr_t)dst, 16, vo, 0, 0, 0);
      if constexpr (G::ROW == 2048) __builtin_amdgcn_raw_ptr_buffer_load_lds(rX, (lptr_t)(dst + 1024), 16, vo, 1024, 0, 0);
      vo += pitch;
    }
  };

  typedef u32x4_t Frags[NI];
  const int frag_vo = (threadIdx.x & 63) * 16;
  auto load_frag = [&](const __amdgpu_buffer_rsrc_t& r, int s, int i) {
    return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, frag_vo, woff + s * G::STEP + i * 1024, 0));
  };
  f32x4_t acc[NI][TJ];
  Frags wb[2];
  u32x4_t fb[2][TJ];
  // One sub-step: NI x TJ MFMAs (the first of a product starts from 0: no pass that clears the accumulators, and
  // none of the wait states that a just-written addend needs, see GemmTile::settle); the token fragments of the next sub-step are read behind the first of them, and
  // each parameter fragment is replaced, one MFMA after its last use, by that of sub-step `ns` of stream `nr`.
  auto substep = [&](auto first_tag, const char* xrow, int s, int buf, bool more, bool refill, const __amdgpu_buffer_rsrc_t& nr, int ns) {
    const char* const xn = xrow + (s + 1) * 64;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        if constexpr (decltype(first_tag)::value)
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[i][j]) : "v"(wb[buf][i]), "v"(fb[buf][j]));
        else
          Elem<bf16_tag>::mma(acc[i][j], reinterpret_cast<const u32x4_t(&)[1]>(wb[buf][i]),
                              reinterpret_cast<const u32x4_t(&)[1]>(fb[buf][j]));
        if (more && i < 2 && (TJ <= 4 || j % 2 == i)) {
          // TJ reads over the first two rows of blocks
          if (TJ > 4 || (i == 0)) fb[buf ^ 1][j] = *reinterpret_cast<const u32x4_t*>(xn + j * 16 * G::PITCH);
        }
        if (refill && j == 0 && i > 0) wb[buf][i - 1] = load_frag(nr, ns, i - 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (refill) wb[buf][NI - 1] = load_frag(nr, ns, NI - 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // acc = X W for one stream; with `chain`, the first two sub-steps of the next stream are on their way at the end
  auto product = [&](const __amdgpu_buffer_rsrc_t& r, bool chain, const __amdgpu_buffer_rsrc_t& next, auto&& per_substep) {
    const int l = lane_id();
    const char* const xrow = smem + (l & 15) * G::PITCH + (l >> 4) * 16;
#pragma unroll
    for (int j = 0; j < TJ; ++j) fb[0][j] = *reinterpret_cast<const u32x4_t*>(xrow + j * 16 * G::PITCH);
    __builtin_amdgcn_sched_barrier(0);
    substep(std::true_type{}, xrow, 0, 0, true, true, r, 2);
    per_substep(0);
    substep(std::false_type{}, xrow, 1, 1, true, true, r, 3);
    per_substep(1);
    for (int s = 2; s < S - 2; s += 2) {
      substep(std::false_type{}, xrow, s, 0, true, true, r, s + 2);
      per_substep(s);
      substep(std::false_type{}, xrow, s + 1, 1, true, true, r, s + 3);
      per_substep(s + 1);
    }
    substep(std::false_type{}, xrow, S - 2, 0, true, chain, next, 0);
    per_substep(S - 2);
    substep(std::false_type{}, xrow, S - 1, 1, false, chain, next, 1);
    per_substep(S - 1);
    asm volatile("s_nop 15\n\ts_nop 15");   // results are read by ordinary instructions next
  };

  int64_t tile = blockIdx.x;
  const int64_t ntiles = (a.n + G::TOK - 1) / G::TOK;
  load_x(tile * G::TOK);
  for (; tile < ntiles; tile += gridDim.x) {
    const int64_t t0 = tile * G::TOK;
    // the first fragments are requested here and not under the previous tile's softmax, which needs the registers (kept across
    // it, 64 a lane at d = 1024, some spill, and each reload waits for everything in flight: 1164 us for 262144 tokens instead of 982)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      wb[0][i] = load_frag(rU, 0, i);
      wb[1][i] = load_frag(rU, 1, i);
    }
    __builtin_amdgcn_s_waitcnt(wait_vm(2 * NI));   // the token rows have landed
    __syncthreads();

    // ---- x~ = x U
    product(rU, true, rW, [](int) {});
    lds_barrier();   // every wavefront has read its last token fragments
    // rounded to bf16 into the place of x; blocks i, i + 1 are 8 consecutive columns
    {
      const int l = lane_id();
      char* const dst = smem + (l & 15) * G::PITCH + (w * (G::D / NW) + (l >> 4) * (G::D / (4 * NW))) * 2;
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; i += 2) {
          typedef __attribute__((ext_vector_type(8))) float f32x8_t;
          const f32x4_t u = acc[i][j], v = acc[i + 1][j];
          const f32x8_t f = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
          *reinterpret_cast<bf16x8_t*>(dst + 16 * j * G::PITCH + 8 * i) = __builtin_convertvector(f, bf16x8_t);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    lds_barrier();

    // ---- x~ W, with x~ streamed out to memory meanwhile
    const int l2 = lane_id();
    const uint32_t xt0 = (uint32_t)t0 * G::ROW + l2 * 16;
    product(rW, false, rU, [&](int s) {
      constexpr int kEvery = S > G::PIECES ? S / G::PIECES : 1;   // sub-steps a piece
      if (s % kEvery != 0) return;
#pragma unroll
      for (int u = 0; u < (G::PIECES > S ? G::PIECES / S : 1); ++u) {
        const int p = s * G::PIECES / S + u;
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(smem + piece_row(p) * G::PITCH + piece_col(p) + l2 * 16);
        __builtin_amdgcn_raw_buffer_store_b128(v, rXt, xt0 + piece_row(p) * G::ROW + piece_col(p), 0, 0);
      }
    });
    lds_barrier();   // x~ has been read by everybody: its place takes the next tile's rows
    if (tile + gridDim.x < ntiles) load_x((tile + gridDim.x) * G::TOK);

    // ---- softmax, cumulative mask, count
    const int l3 = lane_id();
    const int q = l3 >> 4;
    float* const rt = red + (l3 & 15);   // this lane's tokens: rt[16 j + ...]
    // value of lane `from` (the library's shuffles derive their addresses once for the whole kernel)
    auto of_lane = [](int from, auto v) {
      return __builtin_bit_cast(decltype(v), __builtin_amdgcn_ds_bpermute(from << 2, __builtin_bit_cast(int, v)));
    };
    const int x16 = l3 ^ 16, x32 = l3 ^ 32;
    float mx[TJ];
    {
      // The bias goes onto the finished sums, as in the separate kernels: started from it, the accumulators would round
      // every step of the contraction at the bias's magnitude.  (262144 tokens: 1019 -> 1026 us at d = 1024, 317 -> 313
      // at d = 512, the passes that cleared the accumulators having gone; as fp32 MFMAs of bias * 1 under the maxima of
      // the neighbouring block 1084 and 336.)  Four running maxima per token: a single chain would wait for itself.
      const float* const bp = bias_s + w * (G::D / NW) + q * (G::D / (4 * NW));
      f32x4_t m4[TJ];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const f32x4_t b = *reinterpret_cast<const f32x4_t*>(bp + 4 * i);
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          const f32x4_t z = acc[i][j] + b;
          acc[i][j] = z;
#pragma unroll
          for (int v = 0; v < 4; ++v) m4[j][v] = i == 0 ? z[v] : fmaxf(m4[j][v], z[v]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        float m = fmaxf(fmaxf(m4[j].x, m4[j].y), fmaxf(m4[j].z, m4[j].w));
        m = fmaxf(m, of_lane(x16, m));
        m = fmaxf(m, of_lane(x32, m));
        if (q == 0) rt[w * G::TOK + 16 * j] = m;
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_barrier();
    float own[TJ], above[TJ];   // sums of this lane's run and of the wavefront's runs behind it
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const float* const r = rt + 16 * j;
      mx[j] = r[0];
#pragma unroll
      for (int u = 1; u < NW; ++u) mx[j] = fmaxf(mx[j], r[u * G::TOK]);
      float sum = 0.f;
#pragma unroll
      for (int i = NI - 1; i >= 0; --i) {
        f32x4_t e;
#pragma unroll
        for (int v = 0; v < 4; ++v) e[v] = __builtin_amdgcn_exp2f((acc[i][j][v] - mx[j]) * kLog2e);
        acc[i][j] = e;
        sum += (e.x + e.y) + (e.z + e.w);
      }
      own[j] = sum;
      const float s1 = of_lane(l3 + 16, sum), s2 = of_lane(l3 + 32, sum), s3 = of_lane(l3 + 48, sum);   // modulo 64
      above[j] = (q < 1 ? s3 : 0.f) + (q < 2 ? s2 : 0.f) + (q < 3 ? s1 : 0.f);
      if (q == 0) rt[(NW + w) * G::TOK + 16 * j] = above[j] + sum;
      __builtin_amdgcn_sched_barrier(0);
    }
    lds_barrier();
    int cnt[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const float* const r = rt + NW * G::TOK + 16 * j;
      float tot = 0.f, behind = 0.f;
#pragma unroll
      for (int u = NW - 1; u >= 0; --u) {
        if (u == w) behind = tot;
        tot += r[u * G::TOK];
      }
      const float inv = 1.0f / tot;
      above[j] += behind;
      // The mask does not rise along the run: all of it above the threshold, none of it, or a crossing inside.
      const bool all = above[j] * inv > a.tau, none = !((above[j] + own[j]) * inv > a.tau);
      cnt[j] = all ? 4 * NI : 0;
      if (__any(!all && !none)) {
        int c = 0;
        float run = 0.f;   // blocks behind the current one
#pragma unroll
        for (int i = NI - 1; i >= 0; --i) {
          const f32x4_t e = acc[i][j];
          const float s3 = e.w, s2 = e.z + s3, s1 = e.y + s2, s0 = e.x + s1;
          const float base = above[j] + run;
          c += ((base + s0) * inv > a.tau ? 1 : 0) + ((base + s1) * inv > a.tau ? 1 : 0) +
               ((base + s2) * inv > a.tau ? 1 : 0) + ((base + s3) * inv > a.tau ? 1 : 0);
          run += s0;
        }
        if (!all && !none) cnt[j] = c;
      }
      cnt[j] += of_lane(x16, cnt[j]);
      cnt[j] += of_lane(x32, cnt[j]);
      if (q == 0) reinterpret_cast<int*>(rt)[(2 * NW + w) * G::TOK + 16 * j] = cnt[j];
    }
    lds_barrier();
    if (threadIdx.x < G::TOK && t0 + threadIdx.x < a.n) {
      const int* const r = reinterpret_cast<const int*>(red) + 2 * NW * G::TOK + threadIdx.x;
      int sum = 0;
#pragma unroll
      for (int u = 0; u < NW; ++u) sum += r[u * G::TOK];
      a.k[t0 + threadIdx.x] = sum;
    }
  }
}

template <typename G>
hipError_t launch(const KvGateArgs& a, hipStream_t s) {
  const int64_t tiles = (a.n + G::TOK - 1) / G::TOK;
  const int64_t cus = device_compute_units();
  hipError_t e = allow_lds<kv_gate_kernel<G>>(G::LDS_BYTES);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kv_gate_kernel<G>, dim3((unsigned)(tiles < cus ? tiles : cus)), dim3(64 * G::NW), G::LDS_BYTES, s, a);
  return hipGetLastError();
}

}  // namespace

bool kv_gate_fits(int dtype, int64_t n, int d, int64_t ldx) {
  // x is one buffer with 32-bit offsets: its extent below 2^31 bytes, and 128 rows more below 2^32
  return dtype == LMHEAD_BF16 && (d == 1024 || d == 512) && n >= kKvGateFrom &&
         (n * ldx) * 2 < (1ll << 31) && 128 * ldx * 2 < (1ll << 30);
}

hipError_t launch_kv_gate(const KvGateArgs& a, int d, hipStream_t s) {
  return d == 1024 ? launch<Gate<1024 / (16 * kKvGateWaves), 4>>(a, s) : launch<Gate<512 / (16 * kKvGateWaves), 8>>(a, s);
}

}  // namespace lmhead
