"""GPU: conjugate-gradient scalars formed by the vector kernels from the partial sums, at the sizes where
the sums move to a launch of their own, and with one element more than a chunk."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_02401_amd.solver import tikhonov_pcg
from tests.gpu_util import env, rel_l2, say

pytestmark = pytest.mark.gpu

# FP32 operator applications (~1e-6 relative) times the preconditioned condition number (<= 11 here)
PCG_TOL = 1e-4


def _pcg64(p, mask, order, levels, s, alpha, iters):
    p, mask = p.astype(np.float64), mask.astype(np.float64)
    r = mask * p
    x = np.zeros_like(r)
    z = oracle.matern_cov_apply(r, order, levels, s)
    d, rz = z.copy(), np.sum(r * z)
    for _ in range(iters):
        if np.sum(r * r) <= 1e-28 * np.sum((mask * p) ** 2):
            break  # solved: the identity operator (levels = 0) leaves two eigenvalues
        ad = mask * d + alpha * oracle.matern_cov_apply(d, order, levels, -s)
        a = rz / np.sum(d * ad)
        x += a * d
        r = r - a * ad
        z = oracle.matern_cov_apply(r, order, levels, s)
        rz, old = np.sum(r * z), rz
        d = z + rz / old * d
    return x


# 1024 chunks of an instance are summed in place, more by k_cg_reduce: 2^22 elements is the line for
# both the element-wise partials (chunks of 4096) and, at 512 elements a tile, 2^19 for the fused ones
@pytest.mark.parametrize("fused", ["", "0"])
@pytest.mark.parametrize("shape,order,levels,iters", [
    ((3, 25, 41), 2, 0, 5), ((2, 32, 36), 3, 2, 6), ((1, 1032, 512), 2, 2, 3), ((1, 1028, 4096), 1, 2, 2)])
def test_pcg_iterates_match_64_bits(fused, shape, order, levels, iters):
    gen = np.random.default_rng(51)
    p = (np.cumsum(gen.standard_normal(shape), axis=-1) / 4.0).astype(np.float32)
    mask = (gen.random(shape) < 0.3).astype(np.float32)
    say("pcg parts", shape, order, levels, iters, fused)
    with env(ESWAVE_CG_FUSED=fused):
        x, info = tikhonov_pcg(torch.from_numpy(p).cuda(), torch.from_numpy(mask).cuda(), 2, order, levels, 1.0, 0.1,
                               iters=iters, rtol=0.0)
    # a residual of exactly zero ends the solve at the next look (every fourth iteration)
    assert info["iterations"] == iters or (levels == 0 and float(info["rel_residual"].max()) == 0.0)
    for b in range(shape[0]):
        assert rel_l2(x[b].cpu().numpy(), _pcg64(p[b], mask[b], order, levels, 1.0, 0.1, iters)) <= PCG_TOL, b
