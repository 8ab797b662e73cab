"""Tiles that hold five K-steps of 64 values in LDS (each has a compute unit for itself): contractions around the periods of the
unrolled loop, edges 64 and 128, ragged rows of every length; and the sizes next to them that take the ring."""
import pytest

pytestmark = pytest.mark.gpu


# 16 to 21 K-steps, sizes above those that the few-token kernel takes, with a last token tile past n; 15 K-steps; two tiles to a unit;
# the most tokens that the few-token kernel takes and one more
@pytest.mark.parametrize("n,d", [(1001, 1024), (540, 1088), (500, 1152), (481, 1216), (451, 1280), (421, 1344),
                                 (4001, 1024), (2201, 1088), (1501, 1152), (1901, 1280), (1301, 1344), (900, 960), (1101, 1024),
                                 (256, 1024), (257, 1024), (128, 2048), (129, 2048)])
def test_gate_reconstruction_and_dx(n, d):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + d)
    bf, f32 = dict(dtype=torch.bfloat16, device="cuda"), dict(device="cuda")

    def param(t):     # NaN right behind it
        buf = torch.full((d * d + 65536,), float("nan"), **bf)
        buf[:d * d] = t.flatten()
        return buf[:d * d].view(d, d)
    Q = torch.linalg.qr(torch.randn(d, d, generator=g, **f32))[0]
    U, Ui, W = param(Q), param(Q.t()), param(1.5 * torch.randn(d, d, generator=g, **f32))
    b = torch.randn(d, generator=g, **f32)
    x = torch.randn(n, d, generator=g, **f32).to(torch.bfloat16)
    gx = torch.randn(n, d, generator=g, **f32).to(torch.bfloat16)
    desc = L.make_kv_desc(n, d, "bf16")
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    xt, xhat, xbar, dx = (torch.full((n, d), 3.0, **bf) for _ in range(4))
    k = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    m = torch.full((n, d), 3.0, **f32)
    L.dynakv_gate(desc, x, U, W, b, 0.1, xt, k, m, xhat, ws)
    want = x.double() @ U.double()
    # one rounding to bf16 of an fp32 sum
    assert bool(((xt.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all())
    p = torch.softmax(xt.double() @ W.double() + b.double(), 1)
    mask = p.flip(1).cumsum(1).flip(1)
    # logits are fp32 sums of d terms of up to about 6: errors of 1e-5, so the mask's are a few of these
    assert float((m.double() - mask).abs().max()) <= 1e-4
    # every length from none to all, in a store laid out tightly
    k = torch.randint(0, d + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
    k[0], k[n - 1] = d, 0
    off = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    packed = torch.full((n * d,), float("nan"), **bf)
    L.dynakv_store(desc, xt, k, 0, off, packed, n * d, ws)
    L.dynakv_reconstruct(desc, packed, n * d, off, k, Ui, xbar, ws)
    assert L.dynakv_check(ws) == 0
    keep = torch.arange(d, device="cuda")[None, :] < k[:, None]
    want = torch.where(keep, xt.double(), 0.0) @ Ui.double()
    assert bool(((xbar.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all())
    bws = torch.full((L.dynakv_bwd_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    dU, dW, db = (torch.full(s, 3.0, **f32) for s in ((d, d), (d, d), (d,)))
    L.dynakv_gate_bwd(desc, x, U, W, b, xt, gx, None, 0.0, dx, dU, dW, db, bws)
    q = (gx.double() * xt.double()).cumsum(1)
    gl = p * (q - (p * q).sum(1, keepdim=True))
    gxt = gx.double() * mask + gl @ W.double().t()
    # g_l and g_x~ are rounded to bf16 before they are contracted: the bound of test_gpu_dynakv_bwd.py
    for got, ref in ((dx, gxt @ U.double().t()), (dU, x.double().t() @ gxt), (dW, xt.double().t() @ gl), (db, gl.sum(0))):
        assert float((got.double() - ref).norm() / ref.norm()) <= 1e-2
