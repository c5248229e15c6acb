"""GPU: the full bank's coarse kernel (whole instances that fit one work-group) against the FP64 oracle, on
blocks whose rows are and are not whole 16-byte groups, axes shorter than the filter, the largest and the
smallest blocks, with the depth at its maximum: analysis, synthesis and the squared norm."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_02401_amd as es
from tests.gpu_util import ORACLE_OPS, TOL, rel_l2, say

pytestmark = pytest.mark.gpu

SHAPES = [(8,), (36,), (2,), (4096,), (64, 64), (4, 2048), (12, 20), (6, 10), (64, 128), (90, 90), (2, 4), (40, 24),
          (16, 16, 16), (4, 8, 12), (20, 20, 20), (8, 32, 32), (2, 2, 6), (24, 8, 40)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("order", [1, 2, 4, 7, 8])
def test_coarse_blocks(shape, order):
    levels = 0
    while all(v % 2 ** (levels + 1) == 0 for v in shape):
        levels += 1
    say("fb coarse", shape, order, levels)
    x = np.random.default_rng(sum(shape) + order).standard_normal((3,) + shape).astype(np.float32)
    xt = torch.from_numpy(x).cuda()
    for op in (0, 1):
        y = es.apply_op(op, xt, len(shape), order, levels, 1.0).cpu().numpy()
        for b in range(3):
            ref = ORACLE_OPS[op](x[b].astype(np.float64), order, levels, 1.0)
            assert rel_l2(y[b], ref) < TOL, (op, b)
    n = es.hs_norm_sq(xt, len(shape), order, levels, 1.0).cpu().numpy()
    for b in range(3):
        ref = oracle.hs_norm_sq(x[b].astype(np.float64), order, levels, 1.0)
        assert abs(n[b] - ref) < TOL * ref
