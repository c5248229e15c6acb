"""GPU: the coarse kernels at the limits of their block sizes and of the passes that take a block -- the largest
block of 512 threads and the first above it, rows that are no whole 16-byte groups, lines longer than a
work-group's threads, one coarse level with and without matrix products."""
import numpy as np
import pytest
import torch

import paper_2507_02401_amd as es
from tests.gpu_util import ORACLE_OPS, TOL, rel_l2, say

pytestmark = pytest.mark.gpu
DEV = "cuda"
OPS = [es.es_adjoint, es.es_apply, es.matern_cov_apply, es.matern_sample]

# (shape, levels)
CASES = [((64, 64), 2), ((64, 68), 2), ((128, 100), 2), ((64, 36), 2), ((128, 72), 3), ((88, 92), 2), ((8, 12), 2), ((12, 20), 2),
         ((16, 16, 16), 2), ((16, 16, 20), 2), ((32, 4, 36), 2), ((12, 20, 12), 2), ((2048,), 2), ((2056,), 3), ((6668,), 2),
         ((8192,), 4), ((16384,), 5), ((16380,), 2)]


@pytest.mark.parametrize("order", [1, 3, 5, 8])
@pytest.mark.parametrize("shape,levels", CASES, ids=lambda v: str(v))
def test_small_blocks_match_the_oracle(shape, levels, order):
    x = np.random.default_rng(sum(shape) + order).standard_normal((2,) + shape).astype(np.float32)
    say("coarse sizes", shape, levels, order)
    for fn, ref in zip(OPS, ORACLE_OPS):
        got = fn(torch.from_numpy(x).to(DEV), len(shape), order, levels, 1.0).cpu().numpy()
        for b in range(2):
            err = rel_l2(got[b], ref(x[b].astype(np.float64), order, levels, 1.0))
            assert err < TOL, (fn.__name__, b, err)


def test_batches_larger_than_the_chip_equal_their_instances():
    """More blocks than two per CU: every instance has the bits that it has alone."""
    x = torch.randn((700, 24, 28), generator=torch.Generator(DEV).manual_seed(1), device=DEV)
    say("coarse sizes batch")
    for fn in OPS:
        got = fn(x, 2, 4, 2, 1.0)
        for k in (0, 255, 256, 511, 512, 699):
            assert torch.equal(got[k], fn(x[k].contiguous(), 2, 4, 2, 1.0))
