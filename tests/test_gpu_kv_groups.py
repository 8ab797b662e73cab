"""Store and reconstruction around the sizes where their launches change: one workgroup's tokens, one group of the sort, tiles of the last
group, the most tokens that each form of the store and the one-launch sort take; every length from none to all, and errors in the
first, a middle and the last token."""
import pytest

pytestmark = pytest.mark.gpu


def _problem(n, d, dtype):
    import torch
    import paper_2603_04411_amd as L
    g = torch.Generator(device="cuda").manual_seed(n + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    xt = torch.randn(n, d, generator=g, device="cuda").to(tdt)
    k = torch.randint(0, d + 1, (n,), generator=g, device="cuda", dtype=torch.int32)
    Ui = torch.linalg.qr(torch.randn(d, d, generator=g, device="cuda"))[0].contiguous().to(tdt)   # qr lays it out by columns
    desc = L.make_kv_desc(n, d, dtype)
    ws = torch.full((L.dynakv_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device="cuda")
    off = torch.full((n + 1,), -1, dtype=torch.int64, device="cuda")
    return L, desc, xt, k, Ui, ws, off


@pytest.mark.parametrize("n,d,dtype", [(1, 64, "bf16"), (63, 64, "f32"), (65, 128, "bf16"), (2047, 192, "bf16"), (2049, 1024, "bf16"),
                                       (4097, 320, "f32"), (4500, 1024, "bf16"), (18433, 1024, "bf16"), (20000, 64, "bf16"), (257, 64, "bf16"),
                                       (6144, 64, "f32"), (6145, 64, "bf16"), (16384, 64, "bf16"), (16385, 64, "f32"),
                                       (16385, 2048, "bf16"), (16385, 1984, "bf16"), (16448, 64, "bf16"), (16449, 64, "bf16"),
                                       (32767, 128, "bf16"), (32768, 576, "bf16"), (32769, 128, "f32"), (300, 8192, "f32"),
                                       (24001, 1984, "bf16"), (4200, 2048, "f32")])
def test_store_and_reconstruct(n, d, dtype):
    import torch
    L, desc, xt, k, Ui, ws, off = _problem(n, d, dtype)
    seg = (k.long() + 7) // 8 * 8
    want_off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    want_off[1:] = seg.cumsum(0)
    want_off += 16
    cap = int(want_off[-1])
    packed = torch.full((max(cap, 24),), 5.0, dtype=xt.dtype, device="cuda")
    L.dynakv_store(desc, xt, k, 16, off, packed, cap, ws)
    assert L.dynakv_check(ws) == 0 and torch.equal(off, want_off)
    j = torch.arange(d, device="cuda")
    inside, kept = j[None, :] < seg[:, None], j[None, :] < k[:, None]
    want = torch.full_like(packed, 5.0)
    want[(want_off[:-1, None] + j)[inside]] = torch.where(kept, xt, 0)[inside]
    assert torch.equal(packed, want)
    xbar = torch.full((n, d), 3.0, dtype=xt.dtype, device="cuda")
    ws.fill_(0xFF)
    L.dynakv_reconstruct(desc, packed, cap, off, k, Ui, xbar, ws)
    assert L.dynakv_check(ws) == 0
    want = torch.where(kept, xt, 0).double() @ Ui.double()
    # An fp32 sum of up to d terms with partial sums of up to 4, each rounded by 2^-24 of that: a random walk of d steps, six standard
    # deviations; in bf16 rounded once more.
    bound = 24 * d ** 0.5 * 2.0 ** -24 + (2.0 ** -8 * want.abs() if dtype == "bf16" else 0.0)
    assert bool(((xbar.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("n", [40, 2100, 7000, 32768, 33000])
@pytest.mark.parametrize("where", [0.0, 0.5, 1.0])
def test_errors(n, where):
    import torch
    d = 64
    L, desc, xt, k, Ui, ws, off = _problem(n, d, "bf16")
    k.clamp_(min=1)
    i = int(where * (n - 1))
    cap = int(((k.long() + 7) // 8 * 8).sum())
    packed = torch.empty(n * d + 64, dtype=xt.dtype, device="cuda")
    for bad in (-1, d + 1):
        kb = k.clone()
        kb[i] = bad
        L.dynakv_store(desc, xt, kb, 0, off, packed, packed.numel(), ws)
        assert L.dynakv_check(ws) == -6
    L.dynakv_store(desc, xt, k, 0, off, packed, cap - 8, ws)
    assert L.dynakv_check(ws) == -6
    L.dynakv_store(desc, xt, k, 0, off, packed, cap, ws)
    assert L.dynakv_check(ws) == 0
    good = torch.empty(n, d, dtype=xt.dtype, device="cuda")
    L.dynakv_reconstruct(desc, packed, cap, off, k, Ui, good, ws)
    assert L.dynakv_check(ws) == 0
    for wrong in (-8, 4, cap):       # before the store, off its granules, behind it: that token reads as zeros
        ob, xbar = off.clone(), torch.full_like(good, 3.0)
        ob[i] = wrong
        L.dynakv_reconstruct(desc, packed, cap, ob, k, Ui, xbar, ws)
        assert L.dynakv_check(ws) == -6
        assert bool((xbar[i] == 0).all())
        rest = torch.arange(n, device="cuda") != i
        assert torch.equal(xbar[rest], good[rest])
