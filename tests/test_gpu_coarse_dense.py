"""GPU: the low-pass coarse kernel on 2-D blocks -- its coarsest levels as matrix products (blocks of at
most 32 x 32 samples), the passes around them, and blocks with values that are not finite."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_02401_amd as es
from tests.gpu_util import TOL, rel_l2, say

pytestmark = pytest.mark.gpu
DEV = "cuda"

# (shape, levels): one 16 x 16 tile and four, sides that are no multiples of 16 or 4, stacked rows of one
# level and of five, unequal sides, blocks that reach 32 x 32 after passes, and the largest block
CASES = [((4, 4), 2), ((8, 12), 2), ((16, 16), 4), ((16, 32), 4), ((32, 32), 2), ((32, 32), 5), ((32, 32), 6), ((24, 20), 2),
         ((28, 12), 2), ((32, 8), 3), ((64, 16), 4), ((34, 32), 2), ((40, 24), 3), ((64, 64), 6), ((96, 32), 5), ((36, 100), 2),
         ((128, 128), 7), ((256, 64), 6), ((128, 128), 3), ((64, 256), 2)]


@pytest.mark.parametrize("order", [1, 2, 4, 7, 8])
def test_small_images_match_the_oracle(order):
    for shape, levels in CASES:
        levels = min(levels, *(int(v & -v).bit_length() - 1 for v in shape))
        if levels < 2:
            continue
        x = np.random.default_rng(sum(shape) + order).standard_normal((3,) + shape).astype(np.float32)
        say("coarse dense", shape, order, levels)
        for fn, ref in ((es.matern_cov_apply, oracle.matern_cov_apply), (es.matern_sample, oracle.matern_sample)):
            got = fn(torch.from_numpy(x).to(DEV), 2, order, levels, 1.0).cpu().numpy()
            for b in range(3):
                err = rel_l2(got[b], ref(x[b].astype(np.float64), order, levels, 1.0))
                assert err < TOL, (shape, levels, b, err)


@pytest.mark.parametrize("value", [np.nan, np.inf, 1e38])
def test_values_that_are_not_finite_stay_local(value):
    """db1 (Haar) couples a pixel to its block of 2^(levels - 1) only: no other output may change; every
    instance stands for itself."""
    x = np.random.default_rng(3).standard_normal((2, 64, 64)).astype(np.float32)
    bad = x.copy()
    bad[0, 5, 9] = value
    say("coarse not finite", value)
    clean = es.matern_cov_apply(torch.from_numpy(x).to(DEV), 2, 1, 4, 1.0).cpu().numpy()
    got = es.matern_cov_apply(torch.from_numpy(bad).to(DEV), 2, 1, 4, 1.0).cpu().numpy()
    assert np.array_equal(got[1], clean[1])
    away = np.ones((64, 64), bool)
    away[:8, 8:16] = False
    assert rel_l2(got[0][away], clean[0][away]) < TOL
    if not np.isfinite(value):
        assert not np.isfinite(got[0][:8, 8:16]).any()
