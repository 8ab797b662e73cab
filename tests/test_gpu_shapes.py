"""Sizes at which the kernels' tiling can go wrong: remainders and edges of the splits, the smallest and the largest of a
rule's range, against the fp64 oracle through the C ABI.  Bounds: log-probabilities and entropies are fp32
sums of exact products of the stored values, |error| <= (d + ntiles + 8) * 2^-24 * sum of magnitudes, far below the
1e-4 used here for |z| < 10; gradients carry one bf16 rounding of dZ (2^-9 per element, bf16 storage) and get the
library's 1e-2 relative Frobenius bound, fp32 storage 1e-5."""
import numpy as np
import pytest

import workloads as wl
from oracle import lmhead_oracle as O
from tests.harness import GpuProblem, np64, rel_fro, small_inputs, to_device

pytestmark = pytest.mark.gpu


# vocabulary tiles of 256 merged per wavefront and batch: 1, one per wavefront, one more, a whole batch and its neighbours
@pytest.mark.parametrize("tiles", [1, 15, 16, 17, 127, 128, 129])
@pytest.mark.parametrize("T", [1, 37])
def test_softmax_merge_over_vocabulary_tiles(tiles, T):
    cfg = wl.CONFIGS[1].scaled(P=1, G=3, T=T, d=64, V=256 * tiles - 5, len_lo=1, len_hi=T)
    inp = small_inputs(cfg)
    gp = GpuProblem(cfg, inp["H"], inp["W"], inp["tok"], inp["lens"])
    logp, lse, ent, _, _ = gp.fwd()
    assert gp.check() == 0
    o_lp, o_lse, o_ent = O.lmhead_logprob_fwd(wl.as_f64(inp["H"]), wl.as_f64(inp["W"]), inp["tok"], inp["lens"], cfg.T)
    for got, want in ((logp, o_lp), (lse, o_lse), (ent, o_ent)):
        assert np.abs(np64(got) - want).max() <= 1e-4


def _kv_edges(d, n):
    """Tile edges that the KV products may take."""
    return [e for e in (64, 128, 256) if e == 64 or d > 64]


# token counts at the edges of the rule that picks a tile edge, of the tiles themselves, and of the XCD deal-out
@pytest.mark.parametrize("dtype,d,n", [
    ("bf16", 64, 1), ("bf16", 64, 63), ("bf16", 192, 65), ("bf16", 320, 6553), ("bf16", 320, 6593),
    ("bf16", 448, 16384), ("bf16", 448, 16400), ("bf16", 448, 65537), ("f32", 64, 64), ("f32", 192, 129),
    ("f32", 320, 6600), ("f32", 448, 16390),
    ("bf16", 128, 70001), ("bf16", 320, 40003), ("f32", 128, 70001)])
def test_kv_products_over_tile_edges(dtype, d, n):
    import workloads.dynakv as kv
    from oracle import dynakv_oracle as K
    from tests.harness import KvProblem
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d, dtype=dtype)
    inp = kv.kv_inputs(cfg)
    kp = KvProblem(cfg, inp)
    xt, k, m, _ = kp.gate(cfg.tau)
    off, packed = kp.store(xt, k)
    xbar = kp.reconstruct(packed, int(off[-1].item()), off, k)
    assert kp.check() == 0
    # every tile's first, last and middle rows, and the rows next to a tile boundary
    rows = np.unique(np.clip([v for e in _kv_edges(d, n) for c in (0, 1, n // e // 2, n // e) for v in
                              (c * e - 1, c * e, c * e + e // 2, n - 1)], 0, n - 1))
    f = wl.as_f64
    o = K.gate(f(inp["x"][rows]), f(inp["U"]), f(inp["W"]), inp["b"], cfg.tau, store_dtype=dtype)
    # one bf16 rounding of x~ may fall the other way; the mask moves by the logit that such a step moves (see
    # test_gpu_dynakv.py, whose bounds these are); fp32: sums of d products, d * 2^-24 relative
    ulp, tol_m = (2.0 ** -7, 5e-3) if dtype == "bf16" else (2.0 ** -22, 1e-4)
    got = np64(xt)[rows]
    assert np.all(np.abs(got - o["xt"]) <= ulp * np.abs(o["xt"]) + 1e-6 * np.abs(o["xt"]).max())
    assert np.abs(np64(m)[rows] - o["m"]).max() <= tol_m
    # the reconstruction of what the device stored
    kk = k.cpu().numpy()[rows]
    kept = np.where(np.arange(d)[None, :] < kk[:, None], got, 0.0)
    assert rel_fro(np64(xbar)[rows], kept @ f(inp["U_inv"])) <= (4e-3 if dtype == "bf16" else 1e-5)


# each tile edge of dW / dU with one and several slices, odd token counts and widths that are no multiple of the edge
@pytest.mark.parametrize("dtype,d,n", [("bf16", 64, 1), ("bf16", 192, 515), ("bf16", 1088, 700), ("bf16", 832, 5000),
                                       ("bf16", 1024, 16500), ("bf16", 128, 20001), ("bf16", 320, 9001), ("f32", 64, 3), ("f32", 320, 129), ("f32", 576, 2500)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_kv_parameter_gradients_over_splits(dtype, d, n, accumulate):
    import torch
    import workloads.dynakv as kv
    from tests.harness import KvProblem
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d, dtype=dtype)
    inp = kv.kv_inputs(cfg)
    kp = KvProblem(cfg, inp)
    xt, _, m, _ = kp.gate(cfg.tau)
    g_xhat, _ = kv.upstream(cfg)
    init = None
    if accumulate:
        init = [torch.full(s, 0.25, dtype=torch.float32, device="cuda") for s in ((d, d), (d, d), (d,))]
    dx, dU, dW, db = kp.gate_bwd(xt, to_device(g_xhat), accumulate_into=init)
    assert kp.check() == 0
    # the chain rule in 64 bits from the device's own spectral state and mask
    x, U, W = (torch.from_numpy(wl.as_f64(inp[k])).cuda() for k in ("x", "U", "W"))
    t, gx = xt.double(), torch.from_numpy(wl.as_f64(g_xhat)).cuda()
    p = torch.softmax(t @ W + torch.from_numpy(inp["b"]).cuda().double(), 1)
    mask = p.flip(1).cumsum(1).flip(1)
    r = (gx * t).cumsum(1)
    gl = p * (r - (p * r).sum(1, keepdim=True))
    gxt = gx * mask + gl @ W.t()
    base = 0.25 if accumulate else 0.0
    # bf16: one rounding (2^-9) of the gradients that enter each product; fp32: sums of n or d products
    tol = 1e-2 if dtype == "bf16" else 2e-5
    for got, want in ((dx, gxt @ U.t()), (dU, x.t() @ gxt), (dW, t.t() @ gl), (db, gl.sum(0))):
        off = 0.0 if got is dx else base
        err = (got.double() - off - want).norm() / want.norm()
        # adding to 0.25 in fp32 costs 2^-25 * 0.25 per element
        slack = 2.0 ** -27 * want.numel() ** 0.5 / want.norm() if off else 0.0
        assert err <= tol + slack, (float(err), got.shape)


# one token per block, one more than the blocks there are, shares that differ by one
@pytest.mark.parametrize("n,d", [(1, 64), (2, 128), (2047, 64), (2049, 64), (5000, 192)])
def test_kv_retain_rate_over_block_shares(n, d):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator().manual_seed(n)
    m = torch.rand(n, d, generator=g)
    k = torch.randint(0, d + 1, (n,), generator=g, dtype=torch.int32)
    desc = L.make_kv_desc(n, d, "bf16")
    ws = torch.empty(L.dynakv_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    out, gm = torch.empty(3, device="cuda"), torch.empty(n, d, device="cuda")
    L.dynakv_retain(desc, k.cuda(), m.cuda(), 0.5, out, gm, ws)
    assert L.dynakv_check(ws) == 0
    hard, soft = k.double().mean().item() / d, m.double().mean().item()
    # k is summed exactly; of m at most a few hundred values enter one fp32 sum: well under 256 * 2^-24
    np.testing.assert_allclose(out.cpu().numpy(), [hard, soft, 0.5 * soft ** 2], rtol=1.5e-5)
    np.testing.assert_allclose(gm.cpu().numpy(), soft / (n * d), rtol=1.5e-5)


# packing groups of 16 tokens, scan blocks of 256, the step to a separate prefix sum (1024 blocks) and its second turn (4096),
# counting blocks of 1024, segments of more than one turn of a wavefront
@pytest.mark.parametrize("dtype,d,n", [("bf16", 64, 1), ("bf16", 128, 15), ("bf16", 64, 16), ("f32", 64, 17),
                                       ("bf16", 64, 255), ("bf16", 64, 256), ("bf16", 64, 257), ("f32", 128, 1025),
                                       ("bf16", 64, 2049), ("bf16", 64, 524288), ("bf16", 64, 524300),
                                       ("f32", 576, 2050), ("bf16", 1088, 259), ("bf16", 64, 262144),
                                       ("bf16", 64, 262145), ("bf16", 64, 1048600)])
@pytest.mark.parametrize("off_base", [0, 1000 * 8])
def test_kv_store_and_grouping_over_token_blocks(dtype, d, n, off_base):
    import torch
    import paper_2603_04411_amd as L
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n + d)
    xt = torch.randn(n, d, generator=g, device="cuda").to(tdt)
    k = torch.randint(0, d + 1, (n,), generator=g, dtype=torch.int32, device="cuda")
    desc = L.make_kv_desc(n, d, dtype)
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xA5, dtype=torch.uint8, device="cuda")
    cap = off_base + n * d
    off = torch.full((n + 1,), -1, dtype=torch.int64, device="cuda")
    packed = torch.full((cap,), 5.0, dtype=tdt, device="cuda")
    L.dynakv_store(desc, xt, k, off_base, off, packed, cap, ws)
    assert L.dynakv_check(ws) == 0
    seg = (k.long() + 7) // 8 * 8
    want_off = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), seg.cumsum(0)]) + off_base
    assert torch.equal(off, want_off)
    j = torch.arange(d, device="cuda")[None, :]
    want = torch.full_like(packed, 5.0)
    at = (want_off[:-1, None] + j)
    want[at[j < seg[:, None]]] = torch.where(j < k[:, None], xt, torch.zeros((), dtype=tdt, device="cuda"))[j < seg[:, None]]
    assert torch.equal(packed, want)
    # the identity as U^-1: the reconstruction returns the kept components exactly, every token in its own row
    eye = torch.eye(d, device="cuda").to(tdt)
    xbar = torch.full((n, d), 3.0, dtype=tdt, device="cuda")
    L.dynakv_reconstruct(desc, packed, cap, off, k, eye, xbar, ws)
    assert L.dynakv_check(ws) == 0
    assert torch.equal(xbar, torch.where(j < k[:, None], xt, torch.zeros((), dtype=tdt, device="cuda")))
    # one element too little room: the last non-empty segment is refused and reported, nothing else changes
    if int(seg.sum()) > 0:
        last = int((seg > 0).nonzero()[-1])
        packed.fill_(5.0)
        L.dynakv_store(desc, xt, k, off_base, off, packed, int(want_off[-1]) - 1, ws)
        assert L.dynakv_check(ws) == -6
        want[int(want_off[last]):] = 5.0
        assert torch.equal(packed, want)
        bad = k.clone()
        bad[n // 2] = d + 1
        L.dynakv_store(desc, xt, bad, off_base, off, packed, cap, ws)
        assert L.dynakv_check(ws) == -6


# every tile edge of the logits, dH and dW kernels (token counts and vocabulary sizes that are no multiples of them, tiles that
# lie wholly beyond the vocabulary), one and several slices of dH, one and several vocabulary chunks
@pytest.mark.parametrize("dtype,P,G,T,d,V,chunk", [
    ("bf16", 1, 1, 5, 64, 70, 0), ("bf16", 1, 3, 21, 64, 1025, 256), ("bf16", 1, 3, 64, 128, 4113, 0),
    ("bf16", 1, 7, 27, 576, 17000, 0), ("bf16", 1, 8, 130, 320, 9000, 4096), ("bf16", 2, 8, 64, 256, 33000, 0),
    ("f32", 1, 1, 3, 32, 65, 0), ("f32", 2, 4, 32, 96, 1300, 512), ("f32", 2, 8, 64, 288, 9000, 0),
    ("f32", 1, 4, 40, 1024, 8000, 0)])
@pytest.mark.parametrize("dh16", [False, True])
def test_lm_step_over_tile_edges(dtype, P, G, T, d, V, chunk, dh16):
    cfg = wl.CONFIGS[1].scaled(P=P, G=G, T=T, d=d, V=V, dtype=dtype, len_lo=1, len_hi=T)
    inp = small_inputs(cfg)
    gp = GpuProblem(cfg, inp["H"], inp["W"], inp["tok"], inp["lens"], vocab_chunk=chunk, flags=8 if dh16 else 0)
    gp.ws.fill_(0xFF)                      # scratch that is read before it is written shows up as NaN
    logp, lse, ent, _, _ = gp.fwd()
    g = wl.synthetic_upstream_grad(cfg, inp["lens"])
    dH, dW = gp.bwd(lse, to_device(g))
    assert gp.check() == 0
    H, W = wl.as_f64(inp["H"]), wl.as_f64(inp["W"])
    o_lp, o_lse, o_ent = O.lmhead_logprob_fwd(H, W, inp["tok"], inp["lens"], T)
    for got, want in ((logp, o_lp), (lse, o_lse), (ent, o_ent)):
        assert np.abs(np64(got) - want).max() <= 1e-4
    o_dH, o_dW = O.lmhead_logprob_bwd(H, W, inp["tok"], inp["lens"], T, g.astype(np.float64))
    tol = 1e-2 if dtype == "bf16" else 1e-5
    assert rel_fro(np64(dW), o_dW) <= tol
    assert rel_fro(np64(dH), o_dH) <= (max(tol, 4e-3) if dh16 else tol)   # 2^-9 for the rounding of dH itself


# responses scanned by every workgroup (up to 4096) or by one launch ahead, empty responses, out-of-range ids and lengths
@pytest.mark.parametrize("R,T", [(1, 1), (3, 5), (255, 2), (257, 3), (4096, 2), (4097, 2), (5000, 1)])
def test_index_over_response_counts(R, T):
    import torch
    import paper_2603_04411_amd as L
    d, V = 64, 100
    rng = np.random.default_rng(R)
    lens = rng.integers(0, T + 1, size=R).astype(np.int32)
    lens[0] = T
    tok = rng.integers(0, V, size=R * T).astype(np.int32)
    H = rng.standard_normal((R * T, d)).astype(np.float32)
    W = (rng.standard_normal((V, d)) * 0.1).astype(np.float32)
    cfg = wl.CONFIGS[0].scaled(P=R, G=1, T=T, d=d, V=V, len_lo=0, len_hi=T)
    gp = GpuProblem(cfg, H, W, tok, lens)
    logp, lse, ent, mask, cu = gp.fwd()
    assert gp.check() == 0
    valid = np.arange(T)[None, :] < lens[:, None]
    assert np.array_equal(mask.cpu().numpy(), valid.reshape(-1).astype(np.uint8))
    assert np.array_equal(cu.cpu().numpy(), np.concatenate([[0], np.cumsum(lens)]))
    from tests.harness import assert_index_parity
    assert_index_parity(gp, np.nonzero(valid.reshape(-1))[0], tok)
    z = H.astype(np.float64) @ W.astype(np.float64).T
    o = z[np.arange(R * T), tok] - np.log(np.exp(z).sum(1))
    assert np.abs(np64(logp) - np.where(valid.reshape(-1), o, 0.0)).max() <= 1e-4
    # an id outside the vocabulary on a valid slot is reported by both directions, on a padded one by neither
    g = torch.full((R * T,), 0.5, device="cuda")
    for slot, code in ((0, -6), (int(np.nonzero(~valid.reshape(-1))[0][0]) if (~valid).any() else None, 0)):
        if slot is None:
            continue
        t2 = tok.copy()
        t2[slot] = V
        g2 = GpuProblem(cfg, H, W, t2, lens)
        _, lse2, _, _, _ = g2.fwd()
        assert g2.check() == code
        g2.bwd(lse2, g)
        assert g2.check() == code
    bad = lens.copy()
    bad[R // 2] = T + 1
    g3 = GpuProblem(cfg, H, W, tok, bad)
    g3.fwd()
    assert g3.check() == -6


# the one-kernel gate (large streams, no soft outputs): its smallest size, last tiles of one token and of all but one, strided
# rows, both readings of Eq. 6, thresholds that keep everything and nothing
@pytest.mark.parametrize("d,n,ldx", [(1024, 10240, None), (1024, 10241, None), (512, 10367, None), (1024, 16447, 1088),
                                     (512, 33000, 520)])
@pytest.mark.parametrize("literal", [False, True])
def test_kv_gate_in_one_kernel(d, n, ldx, literal):
    import torch
    import workloads.dynakv as kv
    import paper_2603_04411_amd as L
    from tests.harness import KvProblem
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d)
    kp = KvProblem(cfg, kv.kv_inputs(cfg), flags=L.FLAG_LITERAL_FLIP if literal else 0, ldx=ldx)
    kp.ws.fill_(0xFF)
    xt, k, _, _ = kp.gate(cfg.tau, soft=False)
    xt2, k2, m, _ = kp.gate(cfg.tau)          # the separate kernels, which the oracle tests cover
    assert kp.check() == 0
    # the same bf16 products in the same order of K: the same spectral state
    assert torch.equal(xt, xt2)
    # the mask is the same sum of the same exponentials in another order (<= d * 2^-24 relative): a count may differ only
    # where the other path's mask is within that of the threshold
    rows = torch.arange(n, device="cuda")
    for kk in (k, k2):
        assert int(kk.min()) >= 0 and int(kk.max()) <= d
    lo, hi = torch.minimum(k, k2).long(), torch.maximum(k, k2).long()
    differ = (lo != hi).nonzero().flatten()
    eps = 2 * d * 2.0 ** -24
    for r in differ.tolist():
        assert (m[r, lo[r]:hi[r]] - cfg.tau).abs().max() <= eps
    assert differ.numel() <= 1 + n // 1000
    for tau, want in ((-1.0, d), (1.5, 0)):
        _, kt, _, _ = kp.gate(tau, soft=False)
        assert torch.equal(kt, torch.full_like(kt, want))


# the one-kernel gate against 64 bits, up to the benchmark's stream
@pytest.mark.parametrize("n,d", [(10241, 1024), (10367, 512), (262144, 1024), (262143, 512)])
@pytest.mark.parametrize("literal", [False, True])
def test_kv_gate_in_one_kernel_against_64_bits(n, d, literal):
    import torch
    import paper_2603_04411_amd as L
    tau = 0.1
    g = torch.Generator(device="cuda").manual_seed(n + d)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    sigma = torch.arange(1, d + 1, device="cuda").float().pow(-0.5)
    Q = torch.linalg.qr(torch.randn(d, d, generator=torch.Generator().manual_seed(d)))[0].contiguous().cuda()
    x = torch.empty(n, d, dtype=torch.bfloat16, device="cuda")
    for r in range(0, n, 65536):
        x[r:r + 65536] = (randn(min(65536, n - r), d) * sigma) @ Q.t()
    U, W = (Q + 0.02 / d ** 0.5 * randn(d, d)).bfloat16(), (1.5 * randn(d, d)).bfloat16()
    j = torch.arange(d, device="cuda").float()
    b = 6.0 * torch.exp(-((j - 0.35 * d) ** 2) / (2 * (0.12 * d) ** 2))
    desc = L.make_kv_desc(n, d, "bf16", flags=L.FLAG_LITERAL_FLIP if literal else 0)
    xt, k = torch.full_like(x, 3.0), torch.full((n,), -7, dtype=torch.int32, device="cuda")
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    L.dynakv_gate(desc, x, U, W, b, tau, xt, k, None, None, ws)
    assert L.dynakv_check(ws) == 0
    for r in range(0, n, 16384):
        e = min(n, r + 16384)
        want = x[r:e].double() @ U.double()
        # one rounding to bf16, which fp32 sums of d products (d * 2^-24 of the terms' magnitude) may tip the other way
        scale = x[r:e].double().abs() @ U.double().abs()
        assert bool(((xt[r:e].double() - want).abs() <= 2.0 ** -8 * want.abs() + d * 2.0 ** -24 * scale).all())
        z = xt[r:e].double() @ W.double()
        p = torch.softmax(z + b.double(), 1)
        if literal:
            p = p.flip(1)
        m = p.flip(1).cumsum(1).flip(1)
        # fp32 logits: d roundings at the partial sums' magnitude, below 2^6 here, less with their random signs: sqrt(d) 2^-18;
        # the mask moves by at most that, its own sums by d 2^-24
        eps = d ** 0.5 * 2.0 ** -18 + d * 2.0 ** -24
        kk = k[r:e].long()
        assert bool((kk >= (m > tau + eps).sum(1)).all()) and bool((kk <= (m > tau - eps).sum(1)).all())


# the few-token products: one token to a group of 16 and its neighbours, the contraction shared by two to sixteen wavefronts and
# taken in several turns, strided rows
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,d,ldx", [(1, 64, None), (1, 1024, None), (15, 128, 136), (16, 1024, 1032), (17, 576, None),
                                     (33, 1088, None), (240, 1024, None), (8, 2048, None)])
def test_kv_gate_of_few_tokens(dtype, n, d, ldx):
    import workloads.dynakv as kv
    from oracle import dynakv_oracle as K
    from tests.harness import KvProblem
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d, dtype=dtype)
    inp = kv.kv_inputs(cfg)
    kp = KvProblem(cfg, inp, ldx=ldx)
    kp.ws.fill_(0xFF)
    xt, k, m, xhat = kp.gate(cfg.tau)
    assert kp.check() == 0
    f = wl.as_f64
    o = K.gate(f(inp["x"]), f(inp["U"]), f(inp["W"]), inp["b"], cfg.tau, store_dtype=dtype)
    # bounds as in test_kv_products_over_tile_edges
    ulp, tol_m = (2.0 ** -7, 5e-3) if dtype == "bf16" else (2.0 ** -22, 1e-4)
    assert np.all(np.abs(np64(xt) - o["xt"]) <= ulp * np.abs(o["xt"]) + 1e-6 * np.abs(o["xt"]).max())
    assert np.abs(np64(m) - o["m"]).max() <= tol_m
    assert np.abs(np64(xhat) - np64(xt) * np64(m)).max() <= 2.0 ** -8 * np.abs(np64(xt)).max()
    xt2, k2, _, _ = kp.gate(cfg.tau, soft=False)
    assert np.array_equal(np64(xt2), np64(xt)) and np.array_equal(k2.cpu().numpy(), k.cpu().numpy())


# one pass over several weight matrices against separate calls, bit for bit, at sizes where a rule that counted the vocabulary
# rows of all the matrices would take another tile edge than the single call
@pytest.mark.parametrize("dtype,N,V,d", [("bf16", 208, 32000, 64), ("bf16", 520, 8192, 64), ("bf16", 264, 4096, 128),
                                         ("bf16", 60, 16500, 64), ("f32", 8200, 4096, 32), ("f32", 200, 151936, 32)])
def test_multi_policy_pass_is_bit_identical_to_separate_calls(dtype, N, V, d):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(N + V)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    H = torch.randn(N, d, generator=g, device="cuda").to(tdt)
    Ws = [(torch.randn(V, d, generator=g, device="cuda") * 0.1).to(tdt) for _ in range(3)]
    tok = torch.randint(0, V, (N,), generator=g, device="cuda", dtype=torch.int32)
    lens = torch.tensor([N // 2, N // 2 - 3], dtype=torch.int32, device="cuda")
    desc = L.make_desc(1, 2, N // 2, d, V, dtype)
    out = lambda: torch.full((N,), 7.0, device="cuda")  # noqa: E731
    singles = []
    ws = torch.empty(L.workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    for W in Ws:
        o = [out() for _ in range(3)]
        L.lmhead_logprob_fwd(desc, H, W, tok, lens, *o, None, None, ws)
        singles.append(o)
    for npol in (1, 2, 3):
        logps, lse, ent = [out() for _ in range(npol)], out(), out()
        ws = torch.empty(L.multi_workspace_bytes(desc, npol), dtype=torch.uint8, device="cuda")
        L.lmhead_logprob_fwd_multi(desc, H, Ws[:npol], tok, lens, logps, lse, ent, None, None, ws)
        assert all(torch.equal(logps[p], singles[p][0]) for p in range(npol)), npol
        assert torch.equal(lse, singles[0][1]) and torch.equal(ent, singles[0][2]), npol


# vocabulary rows masked with -inf: a run of 256 of them is one tile, or several, that holds nothing; few and many slots
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [40, 1100])
def test_vocabulary_tiles_of_minus_infinity(dtype, T):
    cfg = wl.CONFIGS[1].scaled(P=1, G=2, T=T, d=64, V=1024, dtype=dtype, len_lo=1, len_hi=T)
    inp = small_inputs(cfg)
    H, W = inp["H"].copy(), inp["W"].copy()
    one, ninf = (0x3F80, 0xFF80) if dtype == "bf16" else (1.0, -np.inf)
    H[:, 0] = one
    W[256:512, 0] = ninf
    tok = inp["tok"] % 256
    gp = GpuProblem(cfg, H, W, tok, inp["lens"])
    logp, lse, ent, _, _ = gp.fwd()
    assert gp.check() == 0
    rows = np.r_[0:256, 512:1024]          # what is left of the vocabulary; the ids lie in its first 256
    o = O.lmhead_logprob_fwd(wl.as_f64(H), wl.as_f64(W[rows]), tok, inp["lens"], cfg.T)
    for got, want in zip((logp, lse, ent), o):
        assert np.abs(np64(got) - want).max() <= 1e-4


MASKED = [("bf16", 40, 64, 1024), ("bf16", 200, 64, 16384), ("bf16", 2200, 64, 5000), ("bf16", 40, 1024, 150001), ("bf16", 204, 1024, 150001),
          ("f32", 40, 64, 1024), ("f32", 2200, 64, 16384)]


# the same at every tile edge and in the ranges of a long W, and runs that begin and end inside a tile: a masked row counts for nothing
@pytest.mark.parametrize("runs", ["one tile", "any"])
@pytest.mark.parametrize("dtype,n,d,V", MASKED)
def test_runs_of_minus_infinity(dtype, n, d, V, runs):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + V)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    H = torch.randn(n, d, generator=g, device="cuda").to(tdt)
    W = (0.1 * torch.randn(V, d, generator=g, device="cuda")).to(tdt)
    H[:, 0] = 1.0
    keep = torch.ones(V, dtype=torch.bool, device="cuda")
    for at, length in [(256, 256)] if runs == "one tile" else [(3, 1), (70, 50), (131, 301), (V // 2 - 9, V // 64), (V - 33, 33)]:
        keep[at:at + length] = False
    W[~keep, 0] = -float("inf")
    ids = keep.nonzero().flatten()
    tok = ids[torch.randint(0, len(ids), (n,), generator=g, device="cuda")].int()
    lens = torch.tensor([n], dtype=torch.int32, device="cuda")
    desc = L.make_desc(1, 1, n, d, V, dtype)
    ws = torch.full((L.workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    logp, lse, ent = (torch.full((n,), 7.0, device="cuda") for _ in range(3))
    L.lmhead_logprob_fwd(desc, H, W, tok, lens, logp, lse, ent, None, None, ws)
    assert L.lmhead_check(ws) == 0
    z = H.double() @ W[keep].double().t()
    want = z.logsumexp(1)
    zy = (H.double() * W[tok.long()].double()).sum(1)
    entropy = want - (torch.softmax(z, 1) * z).sum(1)
    # an fp32 sum of d terms, a random walk of roundings by 2^-24 of its partial sums, six standard deviations; the merge of the sums and
    # their logarithm, some roundings of 2^-24 of a figure below 20 each
    bound = 6 * d ** 0.5 * 2.0 ** -24 * float(z.abs().max()) + 32 * 2.0 ** -24 * 20
    assert float((lse.double() - want).abs().max()) <= bound
    assert float((logp.double() - (zy - want)).abs().max()) <= 2 * bound
    assert float((ent.double() - entropy).abs().max()) <= 4 * bound


# many tokens per block of the sum: its error is that of one rounding to fp32, not of a long fp32 chain
@pytest.mark.parametrize("n,d", [(4096, 1024), (16000000, 64)])
def test_kv_retain_rate_of_a_constant_mask(n, d):
    import torch
    import paper_2603_04411_amd as L
    desc = L.make_kv_desc(n, d, "bf16")
    m = torch.full((n, d), 0.1, device="cuda")
    out = torch.empty(3, device="cuda")
    ws = torch.empty(L.dynakv_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    L.dynakv_retain(desc, None, m, 0.5, out, None, ws)
    assert L.dynakv_check(ws) == 0
    want = float(np.float32(0.1))
    # 16 values are added up in fp32 before fp64 takes over (four roundings, 2^-24 each), then one rounding of the result
    assert abs(float(out[1]) - want) <= 5 * 2.0 ** -24 * want


# a bias far above the logits (softmax does not see a common offset): the product is complete before the bias is added, as in
# the separate kernels, so that the logits have one rounding at the bias's magnitude and not one per step of the contraction
@pytest.mark.parametrize("d", [512, 1024])
def test_kv_gate_in_one_kernel_under_a_large_bias(d):
    import torch
    import workloads.dynakv as kv
    from tests.harness import KvProblem
    n = 10300
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d)
    kp = KvProblem(cfg, kv.kv_inputs(cfg))
    kp.b = kp.b + 1.0e5
    _, k, _, _ = kp.gate(cfg.tau, soft=False)
    _, k2, m, _ = kp.gate(cfg.tau)
    assert kp.check() == 0
    lo, hi = torch.minimum(k, k2).long(), torch.maximum(k, k2).long()
    for r in (lo != hi).nonzero().flatten().tolist():
        # equal logits: the two masks are sums of the same exponentials in two orders
        assert (m[r, lo[r]:hi[r]] - cfg.tau).abs().max() <= 2 * d * 2.0 ** -24
