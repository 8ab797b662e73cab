"""Contractions whose operands run along the contraction in memory (W for dH, the hidden states and dZ for dW, both
operands of the gate's parameter gradients): sizes at the edges of their tiles, of their K-steps of 64 rows and of their
2 GiB windows, with NaN wherever a row or column is padding, behind W and the parameters, and in all of the workspace before the
call."""
import numpy as np
import pytest

import workloads.dynakv as kv
from tests.harness import KvProblem, np64, rel_fro, to_device
from tests.test_gpu_dynakv_bwd import _oracle_bwd

pytestmark = pytest.mark.gpu


# bf16: dZ is rounded once (2^-9 relative per element, as uniform noise 1.1e-3 of the result) and everything else summed in fp32;
# fp32: logits of up to 3 with errors of some 1e-6 go through the exponential
TOL_LM = {"bf16": 2.0 ** -8, "f32": 2e-5}


# N, d, V, ldW, vocab_chunk: one K-step and less; tiles 64, 128 and 256 wide; a chunk whose last K-step is past the vocabulary;
# columns past d in the last tile; a W of 2.3 GB (two windows); a dZ of 2.5 GB
@pytest.mark.parametrize("dtype,N,d,V,ldW,chunk", [
    ("bf16", 3, 64, 5, 64, 0), ("bf16", 63, 64, 65, 128, 0), ("bf16", 130, 320, 1000, 320, 256),
    ("bf16", 700, 576, 4099, 640, 1024), ("bf16", 2100, 64, 20001, 64, 0), ("bf16", 300, 1088, 600, 1096, 0),
    ("bf16", 200, 64, 70000, 16384, 0), ("bf16", 8192, 64, 152001, 64, 0),
    ("f32", 3, 32, 5, 32, 0), ("f32", 33, 96, 65, 100, 0), ("f32", 130, 160, 1000, 160, 256), ("f32", 700, 544, 4099, 576, 1024),
    ("f32", 2100, 32, 20001, 32, 0), ("f32", 300, 1056, 600, 1060, 0), ("f32", 200, 32, 70000, 8192, 0),
    ("f32", 4096, 32, 152001, 32, 0)])
def test_dh_and_dw(dtype, N, d, V, ldW, chunk):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(N + V)
    lens = torch.tensor([N, N - N // 3], dtype=torch.int32, device="cuda")
    tdt, wide_t = (torch.bfloat16, torch.float32) if dtype == "bf16" else (torch.float32, torch.float64)
    H = torch.randn(2 * N, d, generator=g, device="cuda").to(tdt)
    H[2 * N - N // 3:] = float("nan")                                   # padding
    wide = torch.full(((V + 256) * ldW,), float("nan"), dtype=tdt, device="cuda")[:V * ldW].view(V, ldW)
    W = wide[:, :d]
    W.copy_(torch.randn(V, d, generator=g, device="cuda") * 0.05)
    tok = torch.randint(0, V, (2 * N,), generator=g, device="cuda", dtype=torch.int32)
    gl = torch.randn(2 * N, generator=g, device="cuda")
    desc = L.make_desc(1, 2, N, d, V, dtype, vocab_chunk=chunk, ldW=ldW)
    ws = torch.full((L.workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    logp, lse = (torch.empty(2 * N, device="cuda") for _ in range(2))
    L.lmhead_logprob_fwd(desc, H, wide, tok, lens, logp, lse, None, None, None, ws)
    ws.fill_(0xFF)
    dH, dW = torch.full((2 * N, d), 7.0, device="cuda"), torch.full((V, d), 7.0, device="cuda")
    L.lmhead_logprob_bwd(desc, H, wide, tok, lens, lse, gl, dH, dW, ws)
    assert L.lmhead_check(ws) == 0
    valid = torch.arange(2 * N, device="cuda") < 2 * N - N // 3
    Hf, Wf, gv, tv = H[valid].to(wide_t), W.to(wide_t), gl[valid].to(wide_t), tok[valid].long()
    wantH, wantW = torch.zeros_like(Hf), torch.zeros_like(Wf)
    for r in range(0, Hf.shape[0], 2048):
        z = Hf[r:r + 2048] @ Wf.t()
        dz = torch.softmax(z, 1).mul_(-gv[r:r + 2048, None])
        dz[torch.arange(dz.shape[0], device="cuda"), tv[r:r + 2048]] += gv[r:r + 2048]
        wantH[r:r + 2048] = dz @ Wf
        wantW += dz.t() @ Hf[r:r + 2048]
    assert bool((dH[~valid] == 0).all())
    assert float((dH[valid] - wantH).norm() / wantH.norm()) <= TOL_LM[dtype]
    assert float((dW - wantW).norm() / wantW.norm()) <= TOL_LM[dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,d", [(1, 64), (63, 64), (65, 192), (257, 320), (1000, 576), (4100, 128), (5000, 1088)])
def test_gate_parameter_gradients(n, d, dtype):
    import torch
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d, dtype=dtype)
    inp = kv.kv_inputs(cfg)
    kp = KvProblem(cfg, inp, ldx=d + 8)
    kp.x[:, d:] = float("nan")
    xt, _, _, _ = kp.gate(cfg.tau, soft=False)
    g_xhat, _ = kv.upstream(cfg, with_g_m=False)
    o = _oracle_bwd(cfg, inp, g_xhat, None, 0.0, "suffix")
    kp.ws_bwd = torch.full((kp.L.dynakv_bwd_workspace_bytes(kp.desc),), 0xFF, dtype=torch.uint8, device="cuda")
    got = kp.gate_bwd(xt, to_device(g_xhat))
    assert kp.check() == 0
    # the bounds of test_gpu_dynakv_bwd.py: g_l and g_x~ are rounded to the storage type before they are contracted
    errs = {name: rel_fro(np64(t), o[name]) for name, t in zip(("dx", "dU", "dW", "db"), got)}
    assert all(np.isfinite(e) and e <= (1e-2 if dtype == "bf16" else 1e-4) for e in errs.values()), errs


# the tiled products, with a last tile past d columns and a last token tile past n: parameters as the caller has them, each with NaN
# right behind it; edges of the gate's and of the reconstruction's tiles in bf16, then in fp32 (held by test_host_tiles.py; 256 wide
# ones are in test_gpu_deep_tiles.py)
EDGES = {(8300, 64): (64, 64, 64, 64), (1100, 576): (64, 64, 64, 64), (2200, 1088): (128, 128, 128, 128),
         (9000, 320): (128, 128, 128, 128), (33000, 576): (128, 128, 64, 128)}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,d", list(EDGES))
def test_gate_and_reconstruction(n, d, dtype):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def param(t):
        buf = torch.full((d * d + 65536,), float("nan"), dtype=tdt, device="cuda")
        buf[:d * d] = t.flatten()
        return buf[:d * d].view(d, d)
    Q = torch.linalg.qr(torch.randn(d, d, generator=g, device="cuda"))[0]
    U, Ui, W = param(Q), param(Q.t()), param(1.5 * torch.randn(d, d, generator=g, device="cuda"))
    b = torch.randn(d, generator=g, device="cuda")
    x = torch.randn(n, d, generator=g, device="cuda").to(tdt)
    desc = L.make_kv_desc(n, d, dtype)
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    xt, xhat, xbar = (torch.full((n, d), 3.0, dtype=tdt, device="cuda") for _ in range(3))
    k = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    m = torch.full((n, d), 3.0, device="cuda")
    L.dynakv_gate(desc, x, U, W, b, 0.1, xt, k, m, xhat, ws)
    want = x.double() @ U.double()
    # one rounding to bf16 of an fp32 sum
    assert bool(((xt.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all())
    p = torch.softmax(xt.double() @ W.double() + b.double(), 1)
    # logits are fp32 sums of d terms of up to about 6: errors of 1e-5, so the mask's are a few of these
    assert float((m.double() - p.flip(1).cumsum(1).flip(1)).abs().max()) <= 1e-4
    assert torch.equal(k, (m > 0.1).sum(1, dtype=torch.int32))
    off = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    packed = torch.full((n * d,), float("nan"), dtype=tdt, device="cuda")
    L.dynakv_store(desc, xt, k, 0, off, packed, n * d, ws)
    L.dynakv_reconstruct(desc, packed, n * d, off, k, Ui, xbar, ws)
    assert L.dynakv_check(ws) == 0
    keep = torch.arange(d, device="cuda")[None, :] < k[:, None]
    want = torch.where(keep, xt.double(), 0.0) @ Ui.double()
    assert bool(((xbar.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all())
