"""GPU: finite values near the FP32 range in the coarse levels of 2-D images.  The matrix products of the coarsest
levels sum columns before rows, so they can overflow where the level passes do not; such blocks have to
take the passes, and an overflow of the passes stays with the outputs that depend on it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_02401_amd as es
from tests.gpu_util import TOL, rel_l2, say

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _cov(x, order, levels, s=1.0):
    return es.matern_cov_apply(torch.from_numpy(x).to(DEV), 2, order, levels, s).cpu().numpy()


@pytest.mark.parametrize("shape,levels", [((32, 32), 4), ((16, 16), 4), ((8, 16), 3), ((64, 64), 5), ((128, 128), 6)])
def test_neighbours_along_axis_0_stay_finite(shape, levels):
    """db1: the passes filter rows first (3e38 / sqrt(2)), so that the pair's sum stays in range at every level."""
    x = np.zeros((2,) + shape, np.float32)
    x[0, 4:6, 3] = 3e38
    x[1] = np.random.default_rng(5).standard_normal(shape).astype(np.float32)
    say("coarse large axis 0", shape, levels)
    got = _cov(x, 1, levels)
    assert np.isfinite(got).all()
    for b in range(2):
        scale = float(np.abs(x[b]).max())
        ref = oracle.matern_cov_apply(x[b].astype(np.float64) / scale, 1, levels, 1.0)
        assert rel_l2(got[b].astype(np.float64) / scale, ref) < TOL


@pytest.mark.parametrize("pattern", ["pair along axis 1", "corner"])
@pytest.mark.parametrize("shape,levels", [((32, 32), 4), ((64, 64), 4)])
def test_overflow_stays_with_its_outputs(pattern, shape, levels):
    """db1 couples a pixel to its block of 2^(levels - 1): the other outputs are those of an image without the
    large values."""
    x = np.random.default_rng(7).standard_normal((1,) + shape).astype(np.float32)
    bad, q = x.copy(), 2 ** (levels - 1)
    if pattern == "corner":
        n = 16
        bad[0, :n, :n] = 2e38
    else:
        n = q
        bad[0, 4, 2:4] = 3e38
    assert n % q == 0
    say("coarse overflow", pattern, shape, levels)
    clean, got = _cov(x, 1, levels)[0], _cov(bad, 1, levels)[0]
    away = np.ones(shape, bool)
    away[:n, :n] = False
    assert np.isfinite(got[away]).all()
    assert rel_l2(got[away], clean[away]) < TOL


@pytest.mark.parametrize("order", [1, 2, 4, 8])
@pytest.mark.parametrize("s", [-1.5, 1.5])
def test_large_images_match_the_oracle(order, s):
    """The whole image scaled so that its largest value, in or out, is about 1e37: three levels of gain 2 stay
    in range."""
    x = np.random.default_rng(order).standard_normal((32, 32)).astype(np.float32)
    ref = oracle.matern_cov_apply(x.astype(np.float64), order, 4, s)
    scale = 2.0 ** np.floor(np.log2(1e37 / max(np.abs(ref).max(), np.abs(x).max())))
    say("coarse large images", order, s)
    got = _cov((x * np.float32(scale))[None], order, 4, s)[0]
    assert rel_l2(got.astype(np.float64) / scale, ref) < TOL
