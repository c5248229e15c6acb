"""GPU: the transposed non-periodic level that folds the extension's images into its edge tiles, on side
lengths around the tile (32 x 64 in 2-D, 512 in 1-D) and around the shortest length it takes (L - 1
samples; below it the boundary shell runs), against the FP64 oracle."""
import numpy as np
import pytest
import torch

import paper_2507_02401_amd as es
from oracle import symdwt
from tests.gpu_util import TOL, rel_l2, say

pytestmark = pytest.mark.gpu

SIDES = {
    1: ([(1,), (2,), (511,), (512,), (513,)], 3),
    2: ([(3, 3), (33, 65), (34, 66), (31, 63), (64, 130)], 3),
    4: ([(6, 70), (7, 7), (8, 8), (35, 67), (65, 132), (30, 136)], 3),
    6: ([(11, 11), (10, 80), (32, 64), (47, 79), (36, 68)], 2),
    8: ([(15, 15), (14, 15), (15, 64), (16, 16), (17, 18), (33, 65), (33, 66), (34, 67), (35, 68), (47, 77), (48, 128),
         (63, 191), (15,), (16,), (512,), (513,), (514,), (515,), (517,), (527,), (1025,)], 3),
}
CASES = [(shape, order, levels) for order, (shapes, levels) in SIDES.items() for shape in shapes]


@pytest.mark.parametrize("shape,order,levels", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_transposed_levels_around_the_tile(shape, order, levels):
    """The largest error, not only the norm's: an image left out shows on a few edge samples.  A sample
    is a chain of 2 * levels steps of at most 48 products per axis; their rounding stays below
    2e-5 of the largest sample."""
    x = np.random.default_rng(sum(shape) * 17 + order).standard_normal((2,) + shape).astype(np.float32)
    say("sym images", shape, order, levels)
    xt = torch.from_numpy(x).cuda()
    for s in (1.0, -0.5):
        got = es.sym_cov_apply_transpose(xt, len(shape), order, levels, s).cpu().numpy()
        for b in range(2):
            ref = symdwt.sym_cov_apply_transpose(x[b].astype(np.float64), order, levels, s)
            assert rel_l2(got[b], ref) < TOL, b
            assert np.abs(got[b] - ref).max() < 2e-5 * np.abs(ref).max(), b
