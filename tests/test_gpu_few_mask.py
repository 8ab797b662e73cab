"""The gate of few tokens whose mask comes with the logits, next to the sizes where it is a launch of its own: one token, last tiles of one
and of all but one, odd widths, several tiles, both types, with and without soft outputs, a workspace that starts full of ones; calls
one after the other, each against its own tokens."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,d", [(1, 64), (17, 64), (15, 320), (100, 128), (8000, 64), (300, 256), (512, 512), (513, 512), (96, 512), (97, 512),
                                 (85, 768), (86, 768), (32, 1024), (33, 1024), (16, 1088)])
@pytest.mark.parametrize("literal", [False, True])
def test_mask_with_the_logits(dtype, n, d, literal):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n * d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    f32 = dict(device="cuda")
    U = (torch.randn(d, d, generator=g, **f32) / d ** 0.5).to(tdt)
    W = (torch.randn(d, d, generator=g, **f32) / d ** 0.5).to(tdt)
    b = torch.randn(d, generator=g, **f32)
    desc = L.make_kv_desc(n, d, dtype, flags=L.FLAG_LITERAL_FLIP if literal else 0)
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    for _ in range(3):
        x = torch.randn(n, d, generator=g, **f32).to(tdt)
        xt, xhat = (torch.full((n, d), 3.0, dtype=tdt, device="cuda") for _ in range(2))
        k, k_soft = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        m = torch.full((n, d), 3.0, **f32)
        L.dynakv_gate(desc, x, U, W, b, 0.3, xt, k, None, None, ws)
        L.dynakv_gate(desc, x, U, W, b, 0.3, xt, k_soft, m, xhat, ws)
        assert L.dynakv_check(ws) == 0
        p = torch.softmax(xt.double() @ W.double() + b.double(), 1)
        p = p.flip(1) if literal else p
        mask = p.flip(1).cumsum(1).flip(1)
        # logits are fp32 sums of d terms with partial sums of up to 4 (six standard deviations of a random walk of roundings), the mask
        # moves by half their span at most; d more roundings in its own sums
        bound = 24 * d ** 0.5 * 2.0 ** -24 + 2 * d * 2.0 ** -24
        assert float((m.double() - mask).abs().max()) <= bound
        assert torch.equal(xhat, (xt.float() * m).to(tdt))
        assert torch.equal(k_soft, (m > 0.3).sum(1, dtype=torch.int32)) and torch.equal(k, k_soft)
