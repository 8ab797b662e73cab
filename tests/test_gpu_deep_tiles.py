"""Tiles that hold five K-steps of 64 values in LDS (each has a compute unit for itself): contractions around the periods of the
unrolled loop, edges 64 and 128, ragged rows of every length; the sizes next to them that take the ring; and 256 wide tiles, with a
last one past d columns and past n tokens."""
import pytest

pytestmark = pytest.mark.gpu

# what the gate's products take, held by test_host_tiles.py: 16 to 21 K-steps, sizes above those that the few-token kernel takes, with a
# last token tile past n; 15 K-steps; two tiles to a unit; the most tokens that the few-token kernel takes and one more
SIZES = {(1001, 1024): "64 deep", (540, 1088): "64 deep", (500, 1152): "64 deep", (481, 1216): "64 deep", (451, 1280): "64 deep",
         (421, 1344): "64 deep", (4001, 1024): "128 deep", (2201, 1088): "128 deep", (1501, 1152): "64 ring",
         (1901, 1280): "128 deep", (1301, 1344): "64 ring", (900, 960): "64 ring", (1101, 1024): "64 ring",
         (256, 1024): "few", (257, 1024): "64 deep", (128, 2048): "few", (129, 2048): "64 deep"}
# the same of 128 wide tiles with 18, 19 and 21 K-steps, and of 256 wide ones (their tokens sorted in groups, and all together)
MORE = {("bf16", 1901, 1152): "128 deep", ("bf16", 1801, 1216): "128 deep", ("bf16", 1601, 1344): "128 deep",
        ("bf16", 24001, 1984): "256 ring", ("bf16", 40001, 1984): "256 ring", ("f32", 24001, 1984): "256 ring"}


@pytest.mark.parametrize("n,d", list(SIZES))
def test_gate_reconstruction_and_dx(n, d):
    # logits are fp32 sums of d terms of up to about 6: errors of 1e-5, so the mask's are a few of these
    _gate_and_backward(n, d, "bf16", 1.5)


@pytest.mark.parametrize("dtype,n,d", list(MORE))
def test_more_edges(dtype, n, d):
    # Logits of standard deviation 12, fp32 sums of d terms each rounded by up to 2^-24 of that: a random walk of standard deviation
    # 12 * 2^-24 * (d / 3)^0.5, at most 1.9e-5.  The mask's error is at most half the span of a token's logit errors, i.e. five of these.
    _gate_and_backward(n, d, dtype, 12 / d ** 0.5)


def _gate_and_backward(n, d, dtype, scale):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    st, f32 = dict(dtype=tdt, device="cuda"), dict(device="cuda")
    # an fp32 sum of d terms with partial sums of up to 4 (a random walk of d roundings by 2^-24, six standard deviations), rounded to
    # bf16 once more
    rel, eps = (2.0 ** -8, 1e-5) if dtype == "bf16" else (0.0, 24 * d ** 0.5 * 2.0 ** -24)

    def param(t):     # NaN right behind it
        buf = torch.full((d * d + 65536,), float("nan"), **st)
        buf[:d * d] = t.flatten()
        return buf[:d * d].view(d, d)
    Q = torch.linalg.qr(torch.randn(d, d, generator=g, **f32))[0]
    U, Ui, W = param(Q), param(Q.t()), param(scale * torch.randn(d, d, generator=g, **f32))
    b = torch.randn(d, generator=g, **f32)
    x = torch.randn(n, d, generator=g, **f32).to(tdt)
    gx = torch.randn(n, d, generator=g, **f32).to(tdt)
    desc = L.make_kv_desc(n, d, dtype)
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    xt, xhat, xbar, dx = (torch.full((n, d), 3.0, **st) for _ in range(4))
    k = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    m = torch.full((n, d), 3.0, **f32)
    L.dynakv_gate(desc, x, U, W, b, 0.1, xt, k, m, xhat, ws)
    want = x.double() @ U.double()
    assert bool(((xt.double() - want).abs() <= rel * want.abs() + eps).all())
    p = torch.softmax(xt.double() @ W.double() + b.double(), 1)
    mask = p.flip(1).cumsum(1).flip(1)
    assert float((m.double() - mask).abs().max()) <= 1e-4
    # every length from none to all, in a store laid out tightly
    k = torch.randint(0, d + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
    k[0], k[n - 1] = d, 0
    off = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    packed = torch.full((n * d,), float("nan"), **st)
    L.dynakv_store(desc, xt, k, 0, off, packed, n * d, ws)
    L.dynakv_reconstruct(desc, packed, n * d, off, k, Ui, xbar, ws)
    assert L.dynakv_check(ws) == 0
    keep = torch.arange(d, device="cuda")[None, :] < k[:, None]
    want = torch.where(keep, xt.double(), 0.0) @ Ui.double()
    assert bool(((xbar.double() - want).abs() <= rel * want.abs() + eps).all())
    bws = torch.full((L.dynakv_bwd_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    dU, dW, db = (torch.full(s, 3.0, **f32) for s in ((d, d), (d, d), (d,)))
    L.dynakv_gate_bwd(desc, x, U, W, b, xt, gx, None, 0.0, dx, dU, dW, db, bws)
    q = (gx.double() * xt.double()).cumsum(1)
    gl = p * (q - (p * q).sum(1, keepdim=True))
    gxt = gx.double() * mask + gl @ W.double().t()
    # g_l and g_x~ are rounded to the storage type before they are contracted: the bounds of test_gpu_dynakv_bwd.py
    for got, ref in ((dx, gxt @ U.double().t()), (dU, x.double().t() @ gxt), (dW, xt.double().t() @ gl), (db, gl.sum(0))):
        assert float((got.double() - ref).norm() / ref.norm()) <= (1e-2 if dtype == "bf16" else 1e-4)
