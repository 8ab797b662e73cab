"""The forward of few tokens over a large vocabulary (one range of W's rows per workgroup) at the sizes where it can go wrong: one K-step,
an odd number of them, ranges that end inside a unit of 16 rows, up to 128 tokens, one more, and the most; the calls next to it that take tiles;
several weight matrices."""
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(64, 2359301), (320, 471901), (1024, 150001), (8192, 19457), (2048, 73729)]
STEP_SIZES = [(8192, 19457), (2048, 73729)]


@pytest.mark.parametrize("d,V", SIZES)
@pytest.mark.parametrize("n,valid", [(1, 1), (130, 0), (128, 128), (204, 129), (204, 204), (205, 205)])
def test_few_tokens(d, V, n, valid):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + d)
    H = torch.randn(n, d, generator=g, device="cuda").bfloat16()
    W = [torch.full((V + 2, d + 8), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]   # NaN behind and between rows
    for w in W:
        w[:V, :d] = 0.05 * torch.randn(V, d, generator=g, device="cuda")
    tok = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    tok[0], tok[-1] = V - 1, 0
    lens = torch.tensor([valid], dtype=torch.int32, device="cuda")
    desc = L.make_desc(1, 1, n, d, V, "bf16", ldW=d + 8)
    ws = torch.full((L.multi_workspace_bytes(desc, 2),), 0xFF, dtype=torch.uint8, device="cuda")
    f32 = dict(device="cuda")
    logp, multi = torch.full((n,), 7.0, **f32), [torch.full((n,), 7.0, **f32) for _ in range(2)]
    lse, ent = torch.full((n,), 7.0, **f32), torch.full((n,), 7.0, **f32)
    L.lmhead_logprob_fwd_multi(desc, H, W, tok, lens, multi, lse, ent, None, None, ws)
    assert L.lmhead_check(ws) == 0
    for w, m in zip(W, multi):
        z = H[:valid].double() @ w[:V, :d].double().t()
        want = z.logsumexp(1)
        # an fp32 sum of d terms, a random walk of roundings by 2^-24 of its partial sums, six standard deviations; the merge of the sums
        # and their logarithm, some roundings of 2^-24 each
        bound = 6 * d ** 0.5 * 2.0 ** -24 * float(z.abs().max() if valid else 0) + 32 * 2.0 ** -24 * 20
        L.lmhead_logprob_fwd(desc, H, w, tok, lens, logp, lse, ent, None, None, ws)
        assert torch.equal(logp, m)
        assert float((lse[:valid].double() - want).abs().max() if valid else 0) <= bound
        zy = z.gather(1, tok[:valid, None].long())[:, 0]
        assert float((logp[:valid].double() - (zy - want)).abs().max() if valid else 0) <= 2 * bound
        entropy = want - (torch.softmax(z, 1) * z).sum(1)
        assert float((ent[:valid].double() - entropy).abs().max() if valid else 0) <= 4 * bound
        assert not logp[valid:].any() and not lse[valid:].any() and not ent[valid:].any()
        del z
    off, nbytes = L.binding.workspace_region(desc, 1, L.binding.WS_GATHERED_ID)
    assert torch.equal(ws[off:off + nbytes].view(torch.int32)[:valid], tok[:valid])


@pytest.mark.parametrize("d,V", STEP_SIZES)
@pytest.mark.parametrize("n,valid", [(1, 1), (128, 128), (204, 129), (204, 204)])
def test_backward_after_it(d, V, n, valid):
    """dZ takes tiles also where the forward takes ranges; the workspace is sized for both and starts full of ones each time."""
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + d)
    H = torch.randn(n, d, generator=g, device="cuda").bfloat16()
    H[valid:] = float("nan")
    W = (0.02 * torch.randn(V, d, generator=g, device="cuda")).bfloat16()
    tok = torch.randint(0, V, (n,), generator=g, device="cuda", dtype=torch.int32)
    tok[0] = V - 1
    gl = torch.randn(n, generator=g, device="cuda")
    lens = torch.tensor([valid], dtype=torch.int32, device="cuda")
    desc = L.make_desc(1, 1, n, d, V, "bf16")
    ws = torch.full((L.workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    logp, lse = (torch.full((n,), 7.0, device="cuda") for _ in range(2))
    L.lmhead_logprob_fwd(desc, H, W, tok, lens, logp, lse, None, None, None, ws)
    ws.fill_(0xFF)
    dH, dW = torch.full((n, d), 7.0, device="cuda"), torch.full((V, d), 7.0, device="cuda")
    L.lmhead_logprob_bwd(desc, H, W, tok, lens, lse, gl, dH, dW, ws)
    assert L.lmhead_check(ws) == 0
    Hf, Wf, gv = H[:valid].double(), W.double(), gl[:valid].double()
    dz = torch.softmax(Hf @ Wf.t(), 1).mul_(-gv[:, None])
    dz[torch.arange(valid, device="cuda"), tok[:valid].long()] += gv
    assert not dH[valid:].any()
    # dZ is rounded to bf16: 2^-9 of each element
    for got, want in ((dH[:valid], dz @ Wf), (dW, dz.t() @ Hf)):
        assert float((got.double() - want).norm() / want.norm()) <= 2.0 ** -8
