"""What follows g_x~ in a backward call, in one launch and next to it: tokens that end in the first and the last row of a tile or of a
K-step, slices of which the last is short, odd widths, both tile edges, dx within it and apart, the most slices; and gradients
that are added to what is there."""
import dataclasses

import pytest

import workloads as wl
import workloads.dynakv as kv
from oracle import dynakv_oracle as O
from tests.harness import KvProblem, np64, rel_fro, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,dtype", [(1, 64, "bf16"), (1025, 64, "bf16"), (16383, 64, "bf16"), (16385, 64, "bf16"), (65, 320, "bf16"),
                                       (2305, 1088, "bf16"), (1500, 1408, "bf16"), (3, 2112, "bf16"), (97, 3072, "bf16"), (1, 64, "f32"),
                                       (513, 64, "f32"), (129, 192, "f32"), (1025, 704, "f32"), (577, 960, "f32")])
def test_one_launch_after_g_xt(n, d, dtype):
    import torch
    cfg = dataclasses.replace(kv.KV_CONFIGS[1].scaled(n=n, d=d), dtype=dtype)
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
    for _ in range(2):
        base = [torch.full_like(t, 0.5) for t in got[1:]]
        again = kp.gate_bwd(xt, to_device(g_xhat), accumulate_into=base)
        assert kp.check() == 0
        assert torch.equal(again[0], got[0])
        for a, t in zip(again[1:], got[1:]):
            assert torch.equal(a, t + 0.5)


@pytest.mark.parametrize("n,d,kinds", [(700, 704, {12}), (97, 3072, {10, 12}), (16384, 448, {10, 11}), (300, 192, {12})])
def test_timing_kinds_of_the_launches(n, d, kinds):
    import paper_2603_04411_amd as L
    cfg = kv.KV_CONFIGS[1].scaled(n=n, d=d)
    kp = KvProblem(cfg, kv.kv_inputs(cfg))
    xt, _, _, _ = kp.gate(cfg.tau, soft=False)
    g_xhat = to_device(kv.upstream(cfg, with_g_m=False)[0])
    L.lmhead_timing_enable(True)
    try:
        kp.gate_bwd(xt, g_xhat)
        counts = {kind: L.lmhead_timing_read(kind)[1] for kind in range(14)}
    finally:
        L.lmhead_timing_enable(False)
    assert counts == {kind: int(kind in kinds | {5, 8, 9}) for kind in range(14)}
