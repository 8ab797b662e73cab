"""The gate with token rows far apart (the last token of each of many long sequences): strides on both sides of those from which x is
copied, with NaN between the rows."""
import pytest

pytestmark = pytest.mark.gpu


def _problem(n, d, ldx, dtype):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + d)
    tdt, cuda = torch.bfloat16 if dtype == "bf16" else torch.float32, dict(device="cuda")
    x = torch.full(((n - 1) * ldx + d,), float("nan"), dtype=tdt, **cuda).as_strided((n, d), (ldx, 1))
    x.copy_(torch.randn(n, d, generator=g, **cuda))
    U = torch.linalg.qr(torch.randn(d, d, generator=g, **cuda))[0].contiguous().to(tdt)
    W = (12 / d ** 0.5 * torch.randn(d, d, generator=g, **cuda)).to(tdt)    # logits of standard deviation 12
    b = torch.randn(d, generator=g, **cuda)
    desc = L.make_kv_desc(n, d, dtype, ldx=ldx)
    assert L.dynakv_validate_desc(desc) == 0
    return L, desc, g, x, U, W, b


# one K-step of tokens and less, a last one that is not full; slices and none; 2^23 - 8: the longest stride without a copy, two
# K-steps to a window; 2^24: the first of which no K-step fits a window
@pytest.mark.parametrize("n,d,ldx,dtype", [
    (2, 64, 1 << 24, "bf16"), (70, 64, 1 << 24, "bf16"), (300, 320, (1 << 23) - 8, "bf16"), (300, 320, 1 << 23, "bf16"),
    (260, 1024, (1 << 24) + 64, "bf16"), (16, 1024, 1 << 26, "bf16"), (70, 64, 1 << 24, "f32"), (200, 192, (1 << 23) - 8, "f32"),
    (200, 192, (1 << 23) + 4, "f32"), (150, 1024, 1 << 24, "f32")])
def test_backward(n, d, ldx, dtype):
    import torch
    L, desc, g, x, U, W, b = _problem(n, d, ldx, dtype)
    xt = (x.double() @ U.double()).to(x.dtype)
    gx = torch.randn(n, d, generator=g, device="cuda").to(x.dtype)
    ws = torch.full((L.dynakv_bwd_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    dx = torch.full_like(xt, 3.0)
    dU, dW, db = (torch.full(s, 3.0, device="cuda") for s in ((d, d), (d, d), (d,)))
    L.dynakv_gate_bwd(desc, x, U, W, b, xt, gx, None, 0.0, dx, dU, dW, db, ws)
    assert L.dynakv_check(ws) == 0
    p = torch.softmax(xt.double() @ W.double() + b.double(), 1)
    q = (gx.double() * xt.double()).cumsum(1)
    gl = p * (q - (p * q).sum(1, keepdim=True))
    gxt = gx.double() * p.flip(1).cumsum(1).flip(1) + gl @ W.double().t()
    # the bounds of test_gpu_dynakv_bwd.py: g_l and g_x~ are rounded to the storage type before they are contracted
    for got, ref in ((dx, gxt @ U.double().t()), (dU, x.double().t() @ gxt), (dW, xt.double().t() @ gl), (db, gl.sum(0))):
        assert float((got.double() - ref).norm() / ref.norm()) <= (1e-2 if dtype == "bf16" else 1e-4)


# few tokens (any stride as it is); 64 and 128 wide tiles on both sides of their longest stride
@pytest.mark.parametrize("n,d,ldx,dtype", [
    (16, 1024, 1 << 26, "bf16"), (260, 1024, 17043504, "bf16"), (260, 1024, 17043512, "bf16"), (300, 1024, 1 << 25, "bf16"),
    (400, 1344, 8521736, "f32"), (400, 1344, 8521740, "f32"), (2050, 1024, 8454648, "bf16"), (2050, 1024, 8454656, "bf16")])
def test_gate(n, d, ldx, dtype):
    import torch
    L, desc, g, x, U, W, b = _problem(n, d, ldx, dtype)
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    xt = torch.full((n, d), 3.0, dtype=x.dtype, device="cuda")
    k = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    m = torch.full((n, d), 3.0, device="cuda")
    L.dynakv_gate(desc, x, U, W, b, 0.1, xt, k, m, None, ws)
    assert L.dynakv_check(ws) == 0
    want = x.double() @ U.double()
    # one rounding to bf16 of an fp32 sum
    assert bool(((xt.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all())
    p = torch.softmax(xt.double() @ W.double() + b.double(), 1)
    # Logits are fp32 sums of d terms whose partial sums are of size 12, each rounded by up to 2^-24 of that: a random walk of standard
    # deviation 12 * 2^-24 * (d / 3)^0.5, at most 1.6e-5.  The mask's error is at most half the span of a token's logit errors, i.e. six of
    # these.
    assert float((m.double() - p.flip(1).cumsum(1).flip(1)).abs().max()) <= 1e-4
    assert torch.equal(k, (m > 0.1).sum(1, dtype=torch.int32))
