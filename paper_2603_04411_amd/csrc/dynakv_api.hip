// extern "C" entry points of the KV-compression path: host-side validation, workspace carving and
// kernel sequencing.  Every argument error is returned before anything is enqueued.
#include "dynakv_common.h"

using namespace lmhead;

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool aligned256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }

int validate(const dynakv_desc* d) {
  if (!d) return LMHEAD_E_NULL;
  if (d->n <= 0 || d->d <= 0 || d->d > kKvMaxD || d->d % 64 != 0) return LMHEAD_E_SHAPE;
  if (d->dtype != LMHEAD_F32 && d->dtype != LMHEAD_BF16) return LMHEAD_E_DTYPE;
  if (d->flags & ~(uint32_t)(DYNAKV_FLAG_LITERAL_FLIP | DYNAKV_FLAG_ACCUM_GRAD)) return LMHEAD_E_DTYPE;
  if (d->reserved != 0 || d->ldx < d->d) return LMHEAD_E_SHAPE;
  const int64_t esz = d->dtype == LMHEAD_BF16 ? 2 : 4;
  if ((int64_t)d->n * d->d * esz > ((int64_t)1 << 31) - ((int64_t)1 << 20)) return LMHEAD_E_SHAPE;
  if ((int64_t)d->n > (int64_t)INT32_MAX - 2 * kTile) return LMHEAD_E_SHAPE;
  if ((d->ldx * esz) % 16 != 0) return LMHEAD_E_ALIGN;
  return LMHEAD_OK;
}

struct Ws {
  KvLayout L;
  char* base;
  template <typename T>
  T* at(size_t off) const { return reinterpret_cast<T*>(base + off); }
};

// K-contiguous (transposed) or row-padded copy of a dense d x d parameter matrix, zero up to dp rows of the copy
KvCopy param_copy(const void* in, int d, void* out, int64_t ld_out, int64_t dp, bool transposed) {
  return {in, d, d, transposed ? d : dp, d, (int)(transposed ? dp : d), out, ld_out,
          transposed ? KvCopy::kTransposed : KvCopy::kPlain, 0};
}

// common prologue of the compute entry points
int open_ws(const dynakv_desc* desc, void* ws, size_t ws_bytes, Ws& w) {
  const int rc = validate(desc);
  if (rc != LMHEAD_OK) return rc;
  if (!ws) return LMHEAD_E_NULL;
  if (!aligned256(ws)) return LMHEAD_E_ALIGN;
  w.L = make_kv_layout(desc);
  w.base = static_cast<char*>(ws);
  if (ws_bytes < w.L.total) return LMHEAD_E_WORKSPACE;
  return LMHEAD_OK;
}

}  // namespace

extern "C" {

int dynakv_validate_desc(const dynakv_desc* desc) { return validate(desc); }

size_t dynakv_workspace_bytes(const dynakv_desc* desc) {
  if (validate(desc) != LMHEAD_OK) return 0;
  return make_kv_layout(desc).total;
}

int dynakv_gate(const dynakv_desc* desc, const void* x, const void* U, const void* W, const float* b, float tau,
                void* xt, int32_t* k, float* m, void* xhat, void* ws, size_t ws_bytes, void* stream) {
  Ws w;
  const int rc = open_ws(desc, ws, ws_bytes, w);
  if (rc != LMHEAD_OK) return rc;
  if (!x || !U || !W || !b || !xt || !k) return LMHEAD_E_NULL;
  if (!aligned16(x) || !aligned16(U) || !aligned16(W) || !aligned16(b) || !aligned16(xt) ||
      (m && !aligned16(m)) || (xhat && !aligned16(xhat)))
    return LMHEAD_E_ALIGN;
  const KvLayout& L = w.L;
  hipStream_t s = static_cast<hipStream_t>(stream);
  WsHeader* hdr = w.at<WsHeader>(L.hdr);
  const int dt = desc->dtype;
  const int d = desc->d;

  KvPrepareArgs pa{};
  pa.hdr = hdr;
  if (!m && !xhat && kv_gate_fits(dt, L.n, d, desc->ldx)) {
    // nothing but x~ and k is wanted: one kernel, with the parameter matrices in its fragment order
    const bool literal = (desc->flags & DYNAKV_FLAG_LITERAL_FLIP) != 0;
    pa.job[0] = {U, d, d, d, d, d, w.at<void>(L.UT), 0, KvCopy::kFragments, 0};
    pa.job[1] = {W, d, d, d, d, d, w.at<void>(L.WT), 0, literal ? KvCopy::kFragmentsFlipped : KvCopy::kFragments, 0};
    pa.njobs = 2;
    LM_TRY(launch_kv_prepare(dt, pa, s));
    TimedLaunch tl(4, s);
    LM_TRY(launch_kv_gate({x, desc->ldx, w.at<void>(L.UT), w.at<void>(L.WT), b, L.n, tau, literal ? 1 : 0, xt, k}, d, s));
    return LMHEAD_OK;
  }
  if (kv_few_fits(L.n, d)) {
    KvFewArgs fa{x, desc->ldx, U, (int)L.n, d, xt, nullptr, hdr, false, false};
    {
      TimedLaunch tl(4, s);
      LM_TRY(launch_kv_few(dt, fa, s));
    }
    fa = {xt, d, W, (int)L.n, d, nullptr, w.at<float>(L.logits), nullptr, false, false};
    {
      TimedLaunch tl(5, s);
      LM_TRY(launch_kv_few(dt, fa, s));
    }
    TimedLaunch tl(6, s);
    LM_TRY(launch_kv_mask(dt, w.at<float>(L.logits), b, xt, L.n, d, tau, (desc->flags & DYNAKV_FLAG_LITERAL_FLIP) != 0,
                          k, m, xhat, s));
    return LMHEAD_OK;
  }
  const bool kmajor = k_major(dt == LMHEAD_F32);   // parameters as the caller has them
  if (!kmajor) {
    // K-contiguous copies of the two parameter matrices: UT[j][k] = U[k][j], WT likewise
    pa.job[0] = param_copy(U, d, w.at<void>(L.UT), L.ldT, L.dp, true);
    pa.job[1] = param_copy(W, d, w.at<void>(L.WT), L.ldT, L.dp, true);
    pa.njobs = 2;
    LM_TRY(launch_kv_prepare(dt, pa, s));
  }

  KvGemmArgs ga{};
  ga.mode = 0;
  ga.A = kmajor ? U : w.at<void>(L.UT);
  ga.ldA = kmajor ? d : L.ldT;
  ga.bytesA = (kmajor ? (int64_t)d : L.dp) * ga.ldA * L.esz;
  ga.clear = kmajor;
  ga.B = x;
  ga.ldB = desc->ldx;
  ga.M = d;
  ga.Nn = L.n;
  ga.K = d;
  ga.out_e = xt;
  ga.ldo = d;
  ga.hdr = hdr;
  {
    TimedLaunch tl(4, s);
    LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  ga.mode = 1;
  ga.A = kmajor ? W : w.at<void>(L.WT);
  ga.clear = false;
  ga.B = xt;
  ga.ldB = d;
  ga.out_e = nullptr;
  ga.out_f = w.at<float>(L.logits);
  {
    TimedLaunch tl(5, s);
    LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  {
    TimedLaunch tl(6, s);
    LM_TRY(launch_kv_mask(dt, w.at<float>(L.logits), b, xt, L.n, d, tau,
                          (desc->flags & DYNAKV_FLAG_LITERAL_FLIP) != 0, k, m, xhat, s));
  }
  return LMHEAD_OK;
}

int dynakv_store(const dynakv_desc* desc, const void* xt, const int32_t* k, int64_t off_base, int64_t* off,
                 void* packed, int64_t capacity, void* ws, size_t ws_bytes, void* stream) {
  Ws w;
  const int rc = open_ws(desc, ws, ws_bytes, w);
  if (rc != LMHEAD_OK) return rc;
  if (!xt || !k || !off || !packed) return LMHEAD_E_NULL;
  if (capacity < 0 || off_base < 0 || off_base % DYNAKV_GRANULE != 0) return LMHEAD_E_SHAPE;
  if (!aligned16(xt) || !aligned16(packed) || (reinterpret_cast<uintptr_t>(off) & 7u)) return LMHEAD_E_ALIGN;
  const KvLayout& L = w.L;
  hipStream_t s = static_cast<hipStream_t>(stream);
  WsHeader* hdr = w.at<WsHeader>(L.hdr);
  LM_TRY(launch_kv_store(desc->dtype, xt, k, L.n, desc->d, off_base, off, packed, capacity,
                         w.at<int64_t>(L.blocksum), hdr, s));
  return LMHEAD_OK;
}

int dynakv_reconstruct(const dynakv_desc* desc, const void* packed, int64_t packed_elems, const int64_t* off,
                       const int32_t* k, const void* U_inv, void* xbar, void* ws, size_t ws_bytes, void* stream) {
  Ws w;
  const int rc = open_ws(desc, ws, ws_bytes, w);
  if (rc != LMHEAD_OK) return rc;
  if (!packed || !off || !k || !U_inv || !xbar) return LMHEAD_E_NULL;
  const KvLayout& L = w.L;
  if (packed_elems < 0 || packed_elems * L.esz > ((int64_t)1 << 31) - 256) return LMHEAD_E_SHAPE;
  if (!aligned16(packed) || !aligned16(U_inv) || !aligned16(xbar) || (reinterpret_cast<uintptr_t>(off) & 7u))
    return LMHEAD_E_ALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  WsHeader* hdr = w.at<WsHeader>(L.hdr);
  const int dt = desc->dtype;
  const int d = desc->d;

  // A[j][kk] = U_inv[kk][j]: row j of the copy is output column j, contiguous over the retained index
  KvPrepareArgs pa{};
  pa.hdr = hdr;
  const bool kmajor = k_major(dt == LMHEAD_F32);   // U_inv as the caller has it
  if (!kmajor) {
    pa.job[0] = param_copy(U_inv, d, w.at<void>(L.UiT), L.ldT, L.dp, true);
    pa.njobs = 1;
  }
  pa.count = make_kv_count(k, L.n, d, L.nbuckets, w.at<int32_t>(L.hist));
  LM_TRY(launch_kv_prepare(dt, pa, s));
  LM_TRY(launch_kv_order(dt, pa.count, off, packed_elems * L.esz, L.ncap, w.at<int32_t>(L.order),
                         w.at<uint32_t>(L.pos_off), w.at<int32_t>(L.pos_len), hdr, s));

  KvGemmArgs ga{};
  ga.mode = 2;
  ga.A = kmajor ? U_inv : w.at<void>(L.UiT);
  ga.ldA = kmajor ? d : L.ldT;
  ga.bytesA = (kmajor ? (int64_t)d : L.dp) * ga.ldA * L.esz;
  ga.B = packed;
  ga.bytesB = packed_elems * L.esz;
  ga.M = d;
  ga.Nn = L.n;
  ga.K = d;
  ga.order = w.at<int32_t>(L.order);
  ga.pos_off = w.at<uint32_t>(L.pos_off);
  ga.pos_len = w.at<int32_t>(L.pos_len);
  ga.out_e = xbar;
  ga.ldo = d;
  ga.hdr = hdr;
  {
    TimedLaunch tl(7, s);
    LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  return LMHEAD_OK;
}

int dynakv_retain(const dynakv_desc* desc, const int32_t* k, const float* m, float alpha, float* out, float* g_m,
                  void* ws, size_t ws_bytes, void* stream) {
  Ws w;
  const int rc = open_ws(desc, ws, ws_bytes, w);
  if (rc != LMHEAD_OK) return rc;
  if (!out) return LMHEAD_E_NULL;
  if ((m && !aligned16(m)) || (g_m && !aligned16(g_m))) return LMHEAD_E_ALIGN;
  const KvLayout& L = w.L;
  hipStream_t s = static_cast<hipStream_t>(stream);
  LM_TRY(launch_kv_retain(k, m, L.n, desc->d, alpha, out, g_m, w.at<double>(L.red), w.at<WsHeader>(L.hdr), s));
  return LMHEAD_OK;
}

size_t dynakv_bwd_workspace_bytes(const dynakv_desc* desc) {
  if (validate(desc) != LMHEAD_OK) return 0;
  return make_kv_bwd_layout(desc).total;
}

int dynakv_gate_bwd(const dynakv_desc* desc, const void* x, const void* U, const void* W, const float* b,
                    const void* xt, const void* g_xhat, const float* g_m, float g_m_const, void* dx, float* dU,
                    float* dW, float* db, void* ws, size_t ws_bytes, void* stream) {
  const int rc = validate(desc);
  if (rc != LMHEAD_OK) return rc;
  if (!ws || !x || !U || !W || !b || !xt || !g_xhat || !dx || !dU || !dW || !db) return LMHEAD_E_NULL;
  if (!aligned256(ws)) return LMHEAD_E_ALIGN;
  if (!aligned16(x) || !aligned16(U) || !aligned16(W) || !aligned16(b) || !aligned16(xt) || !aligned16(g_xhat) ||
      (g_m && !aligned16(g_m)) || !aligned16(dx) || !aligned16(dU) || !aligned16(dW) || !aligned16(db))
    return LMHEAD_E_ALIGN;
  const KvBwdLayout L = make_kv_bwd_layout(desc);
  if (ws_bytes < L.total) return LMHEAD_E_WORKSPACE;
  char* const base = static_cast<char*>(ws);
  auto at = [&](size_t off) { return static_cast<void*>(base + off); };
  hipStream_t s = static_cast<hipStream_t>(stream);
  WsHeader* hdr = static_cast<WsHeader*>(at(L.hdr));
  const int dt = desc->dtype;
  const int d = desc->d;
  const bool literal = (desc->flags & DYNAKV_FLAG_LITERAL_FLIP) != 0;
  const bool accum = (desc->flags & DYNAKV_FLAG_ACCUM_GRAD) != 0;

  // Parameter operands of the three token-major products.  Few tokens and bf16: as the caller has them, W is K-major in the
  // logits and K-contiguous, like U, in g_l W^T and g_x~ U^T.  fp32: W^T as a K-contiguous copy, W and U as row-padded ones.
  const bool few = kv_few_fits(L.n, d), kmajor = k_major(dt == LMHEAD_F32);
  KvPrepareArgs pa{};
  pa.hdr = hdr;
  pa.job[0] = param_copy(W, d, at(L.WT), L.ldT, L.dp, true);
  pa.job[1] = param_copy(W, d, at(L.Wp), L.ldT, L.dp, false);
  pa.job[2] = param_copy(U, d, at(L.Up), L.ldT, L.dp, false);
  pa.njobs = 3;
  if (!few && !kmajor) LM_TRY(launch_kv_prepare(dt, pa, s));

  KvGemmArgs ga{};
  ga.mode = 1;
  ga.A = kmajor ? W : at(L.WT);
  ga.ldA = kmajor ? d : L.ldT;
  ga.bytesA = (kmajor ? (int64_t)d : L.dp) * ga.ldA * L.esz;
  ga.clear = kmajor;
  ga.B = xt;
  ga.ldB = d;
  ga.M = d;
  ga.Nn = L.n;
  ga.K = d;
  ga.out_f = static_cast<float*>(at(L.logits));
  ga.ldo = d;
  ga.hdr = hdr;
  {
    TimedLaunch tl(5, s);
    if (few)
      LM_TRY(launch_kv_few(dt, {xt, d, W, (int)L.n, d, nullptr, ga.out_f, hdr, false, false}, s));
    else
      LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  {
    // g_l, and the direct part g_xhat * m of dL/dx~ (into the buffer that the next product adds to)
    TimedLaunch tl(8, s);
    LM_TRY(launch_kv_mask_bwd(dt, static_cast<const float*>(at(L.logits)), b, xt, g_xhat, g_m, g_m_const, L.n, d,
                              literal, at(L.gl), at(L.gxt), static_cast<float*>(at(L.dbpart)), L.nblk, s));
  }
  LM_TRY(launch_kv_sum_rows(static_cast<const float*>(at(L.dbpart)), L.nblk, d, d, db, accum, s));

  // g_x~ += g_l W^T
  ga.mode = 3;
  ga.A = kmajor ? W : at(L.Wp);
  ga.clear = false;
  ga.B = at(L.gl);
  ga.out_f = nullptr;
  ga.out_e = at(L.gxt);
  ga.accumulate = true;
  {
    TimedLaunch tl(9, s);
    if (few)
      LM_TRY(launch_kv_few(dt, {at(L.gl), d, W, (int)L.n, d, at(L.gxt), nullptr, nullptr, true, true}, s));
    else
      LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  // dx = g_x~ U^T
  ga.A = kmajor ? U : at(L.Up);
  ga.B = at(L.gxt);
  ga.out_e = dx;
  ga.accumulate = false;
  {
    TimedLaunch tl(10, s);
    if (few)
      LM_TRY(launch_kv_few(dt, {at(L.gxt), d, U, (int)L.n, d, dx, nullptr, nullptr, true, false}, s));
    else
      LM_TRY(launch_kv_gemm(dt, ga, s));
  }

  // Parameter gradients: contractions over the tokens, cut into ksplit slices of the token range (one: stored directly).
  //   dW[k][j] = sum_t x~[t][k] g_l[t][j];  dU[i][k] = sum_t x[t][i] g_x~[t][k]
  // bf16: the operands as they lie, both gradients in one launch.  fp32: token-contiguous copies of them.
  auto token_copy = [&](const void* src, int64_t ld, size_t to) {
    return KvCopy{src, ld, L.n, L.ncap, d, (int)L.dp, at(to), L.ldK, KvCopy::kTransposed, 0};
  };
  GemmTArgs ta{};
  ta.A = at(L.T2);
  ta.ldA = L.ldK;
  ta.B = at(L.T1);
  ta.ldB = L.ldK;
  ta.M = d;
  ta.n_limit = d;
  ta.K = L.ncap;
  ta.n_tiles_cap = L.dp / kTile;
  ta.hdr = hdr;
  ta.ksplit = L.ksplit;
  ta.edge = L.edge;
  ta.part = L.ksplit > 1 ? static_cast<float*>(at(L.part)) : nullptr;
  ta.part_ld = d;
  ta.part_slice = (int64_t)d * d;
  ta.ldo = d;
  ta.accumulate = accum;
  if (k_major(dt == LMHEAD_F32)) {
    ta.A = at(L.gl);
    ta.A2 = at(L.gxt);
    ta.B = xt;
    ta.B2 = x;
    ta.ldA = d;
    ta.ldB = d;
    ta.ldB2 = desc->ldx;
    ta.K = L.n;
    ta.a_bytes = ta.a2_bytes = ta.b_bytes = L.n * d * 2;
    ta.b2_bytes = ((L.n - 1) * desc->ldx + d) * 2;
    ta.out = dW;
    ta.out2 = dU;
    {
      TimedLaunch tl(11, s);
      LM_TRY(launch_gemm_t(dt, ta, s, 2));
    }
    if (L.ksplit > 1) LM_TRY(launch_kv_sum_rows(ta.part, L.ksplit, ta.part_slice, ta.part_slice, dW, accum, s, dU));
    return LMHEAD_OK;
  }
  ta.ldB2 = L.ldK;
  // one gradient, or both: the second one's operands are in T3, T4
  auto param_grad = [&](const KvPrepareArgs& copies, int kind, float* out, float* out2) -> int {
    {
      TimedLaunch tl(13, s);
      LM_TRY(launch_kv_prepare(dt, copies, s));
    }
    ta.out = out;
    ta.out2 = out2;
    ta.A2 = out2 ? at(L.T4) : nullptr;
    ta.B2 = out2 ? at(L.T3) : nullptr;
    {
      TimedLaunch tl(kind, s);
      LM_TRY(launch_gemm_t(dt, ta, s, 2));
    }
    if (L.ksplit > 1) LM_TRY(launch_kv_sum_rows(ta.part, L.ksplit, ta.part_slice, ta.part_slice, out, accum, s, out2));
    return LMHEAD_OK;
  };
  KvPrepareArgs copies{};
  copies.job[0] = token_copy(xt, d, L.T1);
  copies.job[1] = token_copy(at(L.gl), d, L.T2);
  copies.njobs = 2;
  if (L.pair) {
    copies.job[2] = token_copy(x, desc->ldx, L.T3);
    copies.job[3] = token_copy(at(L.gxt), d, L.T4);
    copies.njobs = 4;
    return param_grad(copies, 11, dW, dU);
  }
  const int prc = param_grad(copies, 11, dW, nullptr);
  if (prc != LMHEAD_OK) return prc;
  copies.job[0] = token_copy(x, desc->ldx, L.T1);
  copies.job[1] = token_copy(at(L.gxt), d, L.T2);
  return param_grad(copies, 12, dU, nullptr);
}

int dynakv_check(void* ws, void* stream) { return lmhead_check(ws, stream); }

}  // extern "C"
