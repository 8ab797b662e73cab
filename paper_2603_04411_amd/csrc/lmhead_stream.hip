// The forward of few tokens (bf16), whose time is one read of W.
//
// The tiles of lmhead_gemm.hip are workgroups of their own: each starts from an empty ring, requests nothing during its epilogue, and
// the last round of them is as good as empty.  Here the vocabulary is cut into one range of rows per compute unit, even to 16
// rows, and a workgroup takes its range through all of d in passes of up to 256 rows (128 from 129 tokens on) as ONE sequence of
// K-steps: the ring never runs dry, and the next rows are on their way under the epilogue of the last ones.  The softmax statistics
// of a range stay in registers until its end, one plane per range: of 151936 rows 256 to merge instead of 1187 or 2374.
//  - W goes past the caches (nt): it is read once, and is larger than they are.
//  - Tall tiles: per byte of W as few bytes of hidden states as fit.  These come from L2 but through the same path
//    (128 x 128 tiles: 141 us, without their requests 121; 256 x 128: 137).
//  - Each range begins at another K-step.  Rows lie a power of two of bytes apart, and ranges that all read the same columns at a
//    time meet on the same memory channels (137 us, now 112).
// Kernel alone, 120 tokens, d 1024 / 2048 / 4096, V 151936: tiles 76 / 156 / 266 us, now 72 / 112 / 212 (4.3 / 5.5 / 5.9 TB/s; a copy
// loop without any arithmetic 63 / 113 / 182 at the same K-steps).  Not kept: W straight into registers in fragment order, whose
// half lines are fetched twice with nt (217 us) and leave L1 late without (156); 256 x 256 tiles (200 us for 200 tokens, now 160).
#include "logits_tile.h"

namespace lmhead {

namespace {

#if !defined(LMHEAD_BF16_BLOCK) || LMHEAD_BF16_BLOCK == 16

// A workgroup's tile, four wavefronts (2 x 2), and the steps of W (X) and of the hidden states (Y) that LDS holds.
template <int BM, int BN, int SX_, int SY_>
struct Stream {
  using G = GemmTile<bf16_tag, BM, BN, 2, 2>;
  static constexpr int SX = SX_, SY = SY_;
  static constexpr int X_SLOT = BM * G::KB, Y_SLOT = BN * G::KB;
  static constexpr int LDS_BYTES = SX * X_SLOT + SY * Y_SLOT;
  static constexpr int X_LD = G::A_LD, Y_LD = G::B_LD, LD = X_LD + Y_LD;   // load instructions per wavefront and step
  // still in flight when a step's successor has to have landed (see stream_rows), and when the first one has to
  static constexpr int YOUNG = SX <= SY ? (SX - 2) * LD : (SY - 2) * LD + X_LD, YOUNG0 = SX <= SY ? (SX - 2) * LD + Y_LD : (SY - 1) * LD;
  static_assert(YOUNG0 < 64 && LDS_BYTES <= 160 * 1024, "one vmcnt covers what is in flight");
};
using Stream128 = Stream<256, 128, 3, 3>;   // up to 128 tokens
using Stream256 = Stream<128, 256, 4, 3>;

// `units` units of 16 rows of W from row `first` on, against BN hidden states, in passes of up to BM rows; tile(acc, m0, m_end) for
// each.  K goes from step k0 round to k0.  Rows from load_end on count as zeros and are not read.  Begins and ends with no wavefront
// using the LDS.
template <typename C, typename Tile>
__device__ inline void stream_rows(const char* __restrict__ W, int64_t pitchW, const char* __restrict__ H, int64_t pitchH, int ksteps, int k0,
                                   int first, int units, int load_end, char* __restrict__ smem, Tile&& tile) {
  using G = typename C::G;
  typedef __attribute__((address_space(3))) void* lptr_t;
  constexpr int TM = G::TM, TN = G::TN;
  const int l = G::lane(), w = G::wave();
  auto rsrc = [](const char* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), 0, 0x7fffffff, 0x00020000);
  };
  constexpr uint32_t kOutside = 0x80000000u;    // an offset outside the buffer: zeros, and no memory is touched
  const int passes = (units + G::BM / 16 - 1) / (G::BM / 16);
  auto pass_row = [&](int p) { return first + 16 * (units * p / passes); };

  // this lane's rows in its wavefront's loads: x_row + 8 q of the W tile, y_row + 8 q of the hidden states
  const int x_row = w * C::X_LD * 8 + (l >> 3), y_row = w * C::Y_LD * 8 + (l >> 3);
  uint32_t offW[C::X_LD], offH[C::Y_LD];
#pragma unroll
  for (int q = 0; q < C::X_LD; ++q) offW[q] = (uint32_t)((x_row + 8 * q) * pitchW) + G::ld_byte(x_row + 8 * q);
#pragma unroll
  for (int q = 0; q < C::Y_LD; ++q) offH[q] = (uint32_t)((y_row + 8 * q) * pitchH) + G::ld_byte(y_row + 8 * q);
  const __amdgpu_buffer_rsrc_t rH = rsrc(H);
  __amdgpu_buffer_rsrc_t rW = rsrc(W);
  int xk = k0, xn = 0, xp = 0, xslot = 0, left = 0;         // the step of W that is requested next, its pass, its rows
  int yk = k0, yslot = 0;
  auto open_pass = [&]() {
    const int m0 = pass_row(xp);
    left = xp < passes ? min(pass_row(xp + 1), load_end) - m0 : 0;
    rW = rsrc(W + (left > 0 ? m0 : 0) * pitchW);
  };
  auto load_x = [&](int q) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rW, (lptr_t)(smem + xslot * C::X_SLOT + (w * C::X_LD + q) * 1024), 16,
                                             x_row < left - 8 * q ? offW[q] : kOutside, xk * G::KB, 0, /*nt*/ 2);
  };
  auto load_y = [&](int q) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rH, (lptr_t)(smem + C::SX * C::X_SLOT + yslot * C::Y_SLOT + (w * C::Y_LD + q) * 1024), 16,
                                             offH[q], yk * G::KB, 0, 0);
  };
  auto next_x = [&]() {
    xslot = xslot + 1 == C::SX ? 0 : xslot + 1;
    xk = xk + 1 == ksteps ? 0 : xk + 1;
    if (++xn == ksteps) {
      xn = 0;
      ++xp;
      open_pass();
    }
  };
  auto next_y = [&]() {
    yslot = yslot + 1 == C::SY ? 0 : yslot + 1;
    yk = yk + 1 == ksteps ? 0 : yk + 1;
  };

  // fragments: row 16 i + l % 16 of the wavefront's rows (tokens), 16-byte chunk 4 sub + l / 16; the swizzle of row 16 i + r is that of
  // r with 2 i added to bits 1 and 2
  const int c = l & 15, at = c * G::KB + (((l >> 4) ^ G::swz(c)) << 4);
  const int at_x = G::wave_m() * G::WM * G::KB + at, at_y = C::SX * C::X_SLOT + G::wave_n() * G::WN * G::KB + at;
  auto frag = [&](int base, int i, int sub) {
    return *reinterpret_cast<const u32x4_t*>(smem + (base ^ (((2 * i & 6) ^ 4 * sub) << 4)) + i * 16 * G::KB);
  };
  u32x4_t fx[2][TM][1], fy[2][TN][1];
  typename G::Acc acc;
  // MFMAs of TM / 2 rows of blocks on fragment set `buf`; behind the first of them the reads of X (rx) or Y of `base`, sub-step `sub`,
  // into set `rbuf`, behind the others half of the loads of X (lx) or Y, as in GemmTile's regions.
  constexpr int RMMAS = TM * TN / 2;
  static_assert(RMMAS >= TM + C::X_LD / 2 && RMMAS >= TM + C::Y_LD / 2, "reads and loads have an MFMA each");
  auto region = [&](int buf, int i0, bool rd, bool rx, int base, int sub, int rbuf, bool lx, int q0) {
    const int reads = rx ? TM : TN, loads = (lx ? C::X_LD : C::Y_LD) / 2, gap = (RMMAS - reads) / loads;
#pragma unroll
    for (int idx = 0; idx < RMMAS; ++idx) {
      Elem<bf16_tag>::mma(acc[i0 + idx / TN][idx % TN], fx[buf][i0 + idx / TN], fy[buf][idx % TN]);
      if (rd && idx < reads) {
        if (rx) fx[rbuf][idx][0] = frag(base, idx, sub); else fy[rbuf][idx][0] = frag(base, idx, sub);
      }
      if (idx >= reads && (idx - reads) % gap == 0 && (idx - reads) / gap < loads) {
        if (lx) load_x(q0 + (idx - reads) / gap); else load_y(q0 + (idx - reads) / gap);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // What the caller has requested for its tiles has to be there: a wait for it inside the loop would be one for the whole ring.
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __builtin_amdgcn_sched_barrier(0);
  open_pass();
#pragma unroll
  for (int j = -(C::SX > C::SY ? C::SX : C::SY); j < 0; ++j) {
    if (j - 1 + C::SX >= 0) {
#pragma unroll
      for (int q = 0; q < C::X_LD; ++q) load_x(q);
      next_x();
    }
    if (j + C::SY >= 0) {
#pragma unroll
      for (int q = 0; q < C::Y_LD; ++q) load_y(q);
      next_y();
    }
  }
  __builtin_amdgcn_s_waitcnt(wait_vm(C::YOUNG0));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  int sx = 0, sy = 0;
  // One step.  Its first half requests X(k + SX - 1), into the place of X(k - 1); behind the hand-over barrier in its middle, when the
  // next step has landed and this one has been read, its second half requests Y(k + SY).  Past the last step the requests go on, to
  // nothing, which keeps the counts.
  auto step = [&](auto more_tag) {
    constexpr bool kMore = decltype(more_tag)::value;   // the pass has another step
    const int bx = at_x + sx * C::X_SLOT, by = at_y + sy * C::Y_SLOT;
    region(0, 0, true, true, bx, 1, 1, true, 0);
    region(0, TM / 2, true, false, by, 1, 1, true, C::X_LD / 2);
    next_x();
    __builtin_amdgcn_s_waitcnt(wait_vm(C::YOUNG));
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    sx = sx + 1 == C::SX ? 0 : sx + 1;
    sy = sy + 1 == C::SY ? 0 : sy + 1;
    region(1, 0, kMore, true, at_x + sx * C::X_SLOT, 0, 0, false, 0);
    region(1, TM / 2, kMore, false, at_y + sy * C::Y_SLOT, 0, 0, false, C::Y_LD / 2);
    next_y();
  };
  for (int p = 0; p < passes; ++p) {
    G::zero(acc);
#pragma unroll
    for (int i = 0; i < TM; ++i) fx[0][i][0] = frag(at_x + sx * C::X_SLOT, i, 0);
#pragma unroll
    for (int j = 0; j < TN; ++j) fy[0][j][0] = frag(at_y + sy * C::Y_SLOT, j, 0);
    G::settle(acc);
    __builtin_amdgcn_sched_barrier(0);
    for (int k = 0; k + 1 < ksteps; ++k) step(std::true_type{});
    step(std::false_type{});
    asm volatile("s_nop 15\n\ts_nop 15");   // results are read by ordinary instructions next
    tile(acc, pass_row(p), pass_row(p + 1));
  }
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  __builtin_amdgcn_s_barrier();
}

// Range `range` of `ranges` of a matrix of `rows` rows, in whole units of 16.
__device__ inline void range_of(int rows, int range, int ranges, int& first, int& units) {
  const int64_t n = (rows + 15) / 16;
  const int u0 = (int)(n * range / ranges);
  first = 16 * u0;
  units = (int)(n * (range + 1) / ranges) - u0;
}

template <typename C>
__device__ inline void fwd_block(const FwdArgs& a, int pol, int range, char* smem) {
  using G = typename C::G;
  const char* Wp = static_cast<const char*>(a.W[0]);
#pragma unroll
  for (int p = 1; p < kMaxPolicies; ++p) Wp = (pol == p) ? static_cast<const char*>(a.W[p]) : Wp;
  float* const zy = a.zy + (size_t)pol * a.Ncap;
  int32_t* const gid = a.gid + (size_t)pol * a.Ncap;
  int tkj[G::TN];
#pragma unroll
  for (int j = 0; j < G::TN; ++j) tkj[j] = a.tok_c[G::n_of(j)];
  const bool want_t = a.want_entropy && pol == 0;
  int first, units;
  range_of(a.V, range, a.ntiles, first, units);
  TileStats<G> stats;
  stats.clear();
  const int ksteps = a.d * 2 / G::KB;
  stream_rows<C>(Wp, a.ldW * 2, static_cast<const char*>(a.Hc), a.ldHc * 2, ksteps, range % ksteps, first, units, a.V, smem,
                 [&](typename G::Acc& acc, int m0, int m_end) {
                   m_end = min(m_end, a.V);
                   int64_t at = 0;
                   asm volatile("" : "+s"(at));   // addresses are formed here and not kept in registers across the loop
                   capture_target<G>(a, acc, tkj, m0, m_end, at, zy, gid);
                   stats.add(acc, a.zscale, m_end - m0 - G::m_base(), m_end - m0 == G::BM, want_t);
                 });
  float* const red = reinterpret_cast<float*>(smem);   // [WGM][BN][3], where the steps were
  stats.to_lds(red);
  stats.store(a, red, a.part + (size_t)pol * 3 * a.ntiles * a.Ncap, range, 0, want_t);
}

__global__ __launch_bounds__(256, 1) void fwd_stream_kernel(FwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int pol = blockIdx.x / a.ntiles, range = blockIdx.x - pol * a.ntiles, nv = a.hdr->nv;
  static_assert(kStreamSlots <= 256, "one block of tokens");
  if (nv > 128)
    fwd_block<Stream256>(a, pol, range, smem);
  else if (nv > 0)
    fwd_block<Stream128>(a, pol, range, smem);
}

#endif

}  // namespace

hipError_t launch_fwd_stream(const FwdArgs& a, hipStream_t s) {
#if !defined(LMHEAD_BF16_BLOCK) || LMHEAD_BF16_BLOCK == 16
  constexpr int kLds = Stream256::LDS_BYTES > Stream128::LDS_BYTES ? Stream256::LDS_BYTES : Stream128::LDS_BYTES;
  hipError_t e = allow_lds<fwd_stream_kernel>(kLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fwd_stream_kernel, dim3((unsigned)(a.ntiles * a.npol)), dim3(256), kLds, s, a);
  return hipGetLastError();
#else
  return hipErrorInvalidValue;   // make_layout does not ask for it
#endif
}

}  // namespace lmhead
