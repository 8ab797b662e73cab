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

  if (!m && !xhat && kv_gate_fits(dt, L.n, d, desc->ldx)) {
    // nothing but x~ and k is wanted: one kernel, with the parameter matrices in its fragment order
    const bool literal = (desc->flags & DYNAKV_FLAG_LITERAL_FLIP) != 0;
    KvPrepareArgs pa{};
    pa.hdr = hdr;
    pa.job[0] = {U, d, w.at<void>(L.Ufrag), false};
    pa.job[1] = {W, d, w.at<void>(L.Wfrag), literal};
    pa.njobs = 2;
    LM_TRY(launch_kv_prepare(L.esz, pa, s));
    TimedLaunch tl(4, s);
    LM_TRY(launch_kv_gate({x, desc->ldx, w.at<void>(L.Ufrag), w.at<void>(L.Wfrag), b, L.n, tau, literal ? 1 : 0, xt, k}, d, s));
    return LMHEAD_OK;
  }
  if (kv_few_fits(dt == LMHEAD_F32, L.n, d)) {
    const bool literal = (desc->flags & DYNAKV_FLAG_LITERAL_FLIP) != 0, one = kv_mask_with_logits(L.esz, L.n, d, m || xhat);
    int32_t* const done = one ? w.at<int32_t>(L.order) : nullptr;
    float* const logits = w.at<float>(L.logits);
    {
      TimedLaunch tl(4, s);
      LM_TRY(launch_kv_few(dt, {x, desc->ldx, U, (int)L.n, d, xt, hdr, done, 0}, s));
    }
    const KvFewMask mask{k, done, b, xt, m, xhat, tau, literal};
    {
      TimedLaunch tl(5, s);
      LM_TRY(launch_kv_few(dt, {xt, d, W, (int)L.n, d, logits, nullptr, nullptr, kFewWide}, s, one ? &mask : nullptr));
    }
    if (!one) {
      TimedLaunch tl(6, s);
      LM_TRY(launch_kv_mask(dt, logits, b, xt, L.n, d, tau, literal, k, m, xhat, s));
    }
    return LMHEAD_OK;
  }
  // rows too far apart for a tile's window: a dense copy, where the logits will be
  const int edge = kv_tile_edge(dt == LMHEAD_F32, 0, d, L.n, d, device_compute_units());
  const bool dense = kv_tiles_need_dense(L.n, edge, desc->ldx, d, L.esz);
  KvGemmArgs ga{};
  ga.mode = 0;
  ga.A = U;
  ga.ldA = d;
  ga.bytesA = (int64_t)d * d * L.esz;
  ga.clear = true;
  ga.B = dense ? w.at<void>(L.logits) : x;
  ga.ldB = dense ? d : desc->ldx;
  ga.M = d;
  ga.Nn = L.n;
  ga.K = d;
  ga.out_e = xt;
  ga.ldo = d;
  ga.hdr = hdr;
  {
    TimedLaunch tl(4, s);
    if (dense) LM_TRY(launch_kv_dense(x, desc->ldx * L.esz, L.n, d * L.esz, w.at<void>(L.logits), s));
    LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  ga.mode = 1;
  ga.A = W;
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

  KvGemmArgs ga{};
  if (kv_group_fits(L.esz, L.n, d)) {
    int32_t* const outside = w.at<int32_t>(L.hist);
    const int edge = kv_tile_edge(dt == LMHEAD_F32, 2, d, L.n, d, device_compute_units());   // of the tiles that follow
    LM_TRY(launch_kv_group(dt, k, off, L.n, d, packed_elems * L.esz, L.nbuckets, edge, w.at<int32_t>(L.order),
                           w.at<uint32_t>(L.pos_off), w.at<int32_t>(L.pos_len), outside, s));
    ga.outside = outside;
    ga.groups = (int)((L.n + kKvGroup - 1) / kKvGroup);
  } else {
    KvPrepareArgs pa{};
    pa.hdr = hdr;
    pa.count = make_kv_count(k, L.n, d, L.nbuckets, w.at<int32_t>(L.hist));
    LM_TRY(launch_kv_prepare(L.esz, pa, s));
    LM_TRY(launch_kv_order(dt, pa.count, off, packed_elems * L.esz, L.ncap, w.at<int32_t>(L.order),
                           w.at<uint32_t>(L.pos_off), w.at<int32_t>(L.pos_len), hdr, s));
  }

  ga.mode = 2;
  ga.A = U_inv;
  ga.ldA = d;
  ga.bytesA = (int64_t)d * d * L.esz;
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

  // the parameters as the caller has them: W is K-major in the logits and K-contiguous, like U, in g_l W^T and g_x~ U^T
  const bool few = kv_few_fits(dt == LMHEAD_F32, L.n, d);
  KvGemmArgs ga{};
  ga.mode = 1;
  ga.A = W;
  ga.ldA = d;
  ga.bytesA = (int64_t)d * d * L.esz;
  ga.clear = true;
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
      LM_TRY(launch_kv_few(dt, {xt, d, W, (int)L.n, d, ga.out_f, hdr, nullptr, kFewWide}, s));
    else
      LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  {
    // g_l, and the direct part g_xhat * m of dL/dx~ (into the buffer that the next product adds to)
    TimedLaunch tl(8, s);
    LM_TRY(launch_kv_mask_bwd(dt, static_cast<const float*>(at(L.logits)), b, xt, g_xhat, g_m, g_m_const, L.n, d,
                              literal, at(L.gl), at(L.gxt), static_cast<float*>(at(L.dbpart)), L.nblk,
                              static_cast<int32_t*>(at(L.done)), L.tail ? (int)kv_tail_counters(d) : 0, s));
  }

  // g_x~ += g_l W^T
  ga.mode = 3;
  ga.A = W;
  ga.clear = false;
  ga.B = at(L.gl);
  ga.out_f = nullptr;
  ga.out_e = at(L.gxt);
  ga.accumulate = true;
  {
    TimedLaunch tl(9, s);
    if (few)
      LM_TRY(launch_kv_few(dt, {at(L.gl), d, W, (int)L.n, d, at(L.gxt), nullptr, nullptr, kFewRows | kFewAdd}, s));
    else
      LM_TRY(launch_kv_gemm(dt, ga, s));
  }
  // dx = g_x~ U^T
  ga.A = U;
  ga.B = at(L.gxt);
  ga.out_e = dx;
  ga.accumulate = false;
  const bool dx_apart = !L.tail || kv_tail_dx_apart(dt == LMHEAD_F32, L.n, d, {L.edge, L.ksplit});
  if (dx_apart) {
    TimedLaunch tl(10, s);
    if (few)
      LM_TRY(launch_kv_few(dt, {at(L.gxt), d, U, (int)L.n, d, dx, nullptr, nullptr, kFewRows}, s));
    else
      LM_TRY(launch_kv_gemm(dt, ga, s));
  }

  // x where it lies, unless its rows are too far apart: then a dense copy in the place of the logits, which are done with
  const bool dense = kv_gradient_needs_dense(desc->ldx);
  // Parameter gradients: contractions over the tokens, both in one launch, cut into ksplit slices of the token range (one:
  // stored directly).  dW[k][j] = sum_t x~[t][k] g_l[t][j];  dU[i][k] = sum_t x[t][i] g_x~[t][k]
  GemmTArgs ta{};
  ta.A = at(L.gl);
  ta.A2 = at(L.gxt);
  ta.ldA = d;
  ta.B = xt;
  ta.B2 = dense ? at(L.logits) : x;
  ta.ldB = d;
  ta.ldB2 = dense ? d : desc->ldx;
  ta.a_bytes = ta.a2_bytes = ta.b_bytes = L.n * d * L.esz;
  ta.b2_bytes = ((L.n - 1) * ta.ldB2 + d) * L.esz;
  ta.M = d;
  ta.n_limit = d;
  ta.K = L.n;
  ta.n_tiles_cap = L.dp / kTile;
  ta.hdr = hdr;
  ta.ksplit = L.ksplit;
  ta.edge = L.edge;
  ta.part = L.ksplit > 1 ? static_cast<float*>(at(L.part)) : nullptr;
  ta.part_ld = d;
  ta.part_slice = (int64_t)d * d;
  ta.out = dW;
  ta.out2 = dU;
  ta.ldo = d;
  ta.accumulate = accum;
  const KvSums sums{static_cast<const float*>(at(L.dbpart)), L.nblk, ta.part, L.ksplit, d, db, dW, dU, accum};
  {
    TimedLaunch tl(L.tail ? 12 : 11, s);
    if (dense) LM_TRY(launch_kv_dense(x, desc->ldx * L.esz, L.n, d * L.esz, at(L.logits), s));
    if (L.tail) {
      if (dx_apart) ga.Nn = 0;
      ta.done = static_cast<int32_t*>(at(L.done));
      LM_TRY(launch_kv_tail(dt, ga, ta, sums, s));
      return LMHEAD_OK;
    }
    LM_TRY(launch_gemm_t(dt, ta, s, 2));
  }
  LM_TRY(launch_kv_sums(sums, s));
  return LMHEAD_OK;
}

int dynakv_check(void* ws, void* stream) { return lmhead_check(ws, stream); }

}  // extern "C"
