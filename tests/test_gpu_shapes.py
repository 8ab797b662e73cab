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
