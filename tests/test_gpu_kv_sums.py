"""The sums of the KV path at the sizes where their launches change: the retain rate around the most values that one workgroup
takes, the gradients' sums where the token range is not cut, cut once and cut often."""
import pytest

import workloads as wl
import workloads.dynakv as kv
from oracle import dynakv_oracle as O
from tests.harness import KvProblem, np64, rel_fro, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d", [(1, 64), (63, 64), (4095, 64), (4096, 64), (4097, 64), (31, 8192), (32, 8192), (33, 8192),
                                 (1535, 64), (1536, 64), (1537, 64), (12, 8192), (13, 8192)])
@pytest.mark.parametrize("have", ["k", "m", "both"])
def test_retain_rate(n, d, have):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n * d)
    desc = L.make_kv_desc(n, d, "f32")
    m = torch.rand(n, d, generator=g, device="cuda") if have != "k" else None
    k = torch.randint(-3, d + 4, (n,), generator=g, device="cuda", dtype=torch.int32) if have != "m" else None
    out, gm = torch.full((3,), 7.0, device="cuda"), torch.full((n, d), 7.0, device="cuda")
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    L.dynakv_retain(desc, k, m, 0.5, out, gm, ws)
    assert L.dynakv_check(ws) == 0
    hard = float(k.clamp(0, d).double().sum()) / (n * d) if k is not None else 0.0
    soft = float(m.double().mean()) if m is not None else 0.0
    # sixteen fp32 additions at most before fp64 takes over, and one rounding of each result
    for got, want in zip(out.tolist(), (hard, soft, 0.5 * soft * soft)):
        assert abs(got - want) <= 8 * 2.0 ** -24 * want
    assert float((gm - 2 * 0.5 * out[1] / (n * d)).abs().max()) <= 4 * 2.0 ** -24 / (n * d)


# slices of the token range, in launches of their own (bf16 from some 16000 tokens on, fp32) and in one with the gradients: none, a few,
# one per workgroup; the most that d = 64 and 128 have, summed by columns, and next to them; accumulated and not
GRADIENTS = [(40, 1088, "bf16"), (700, 576, "bf16"), (2000, 64, "bf16"), (16700, 64, "bf16"), (8300, 128, "bf16"), (4200, 192, "bf16"),
             (16700, 128, "bf16"), (16700, 192, "bf16"), (700, 64, "f32"), (1100, 128, "f32"), (512, 192, "f32"), (300, 256, "f32"),
             (40, 576, "f32"), (2000, 1088, "f32"), (2000, 1280, "f32")]


@pytest.mark.parametrize("n,d,dtype", GRADIENTS)
def test_gradient_sums(n, d, dtype):
    import torch
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d, dtype=dtype)
    inp = kv.kv_inputs(cfg)
    kp = KvProblem(cfg, inp)
    xt, _, _, _ = kp.gate(cfg.tau, soft=False)
    g_xhat, _ = kv.upstream(cfg, with_g_m=False)
    f = wl.as_f64
    o = O.gate_bwd(f(inp["x"]), f(inp["U"]), f(inp["W"]), inp["b"], f(g_xhat), None, order="suffix", store_dtype=cfg.dtype)
    got = kp.gate_bwd(xt, to_device(g_xhat))
    for name, t in zip(("dx", "dU", "dW", "db"), got):
        # bf16: g_l and g_x~ are rounded to 2^-9; fp32: sums of max(n, d) terms, with the cancellation in the mask's gradient
        assert rel_fro(np64(t), o[name]) <= (1e-2 if dtype == "bf16" else 1e-4), name
    base = [torch.full_like(t, 0.5) for t in got[1:]]
    again = kp.gate_bwd(xt, to_device(g_xhat), accumulate_into=base)
    assert kp.check() == 0
    assert torch.equal(again[0], got[0])
    for a, t in zip(again[1:], got[1:]):
        assert torch.equal(a, t + 0.5)
