"""GPU: GMRES steps enqueued without waiting for the host, at the sizes where the chunk of the vector
kernels, the place of the reductions and the 16-byte path change."""
import numpy as np
import pytest
import torch

import oracle
from paper_2507_02401_amd.solver import tikhonov_gmres
from tests.gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu

# FP32 operator applications (~1e-6 relative) through the steps of a system of condition <= 11
GMRES_TOL = 1e-4


def _problem(shape, seed):
    gen = np.random.default_rng(seed)
    p = (np.cumsum(gen.standard_normal(shape), axis=-1) / 4.0).astype(np.float32)
    mask = (gen.random(shape) < 0.3).astype(np.float32)
    return p, mask


# n = 9 x 15 (no multiple of four), one element past a chunk of 1024, one past the small-chunk limit
# 2^19, and more than 256 chunks of 4096 (sums in a launch of their own)
@pytest.mark.parametrize("shape,ndim,order,levels,steps", [
    ((2, 9, 15), 2, 2, 0, 6), ((1, 25, 41), 2, 2, 0, 7), ((3, 32, 36), 2, 3, 2, 15),
    ((1, 728, 724), 2, 2, 2, 5), ((1, 1032, 1024), 2, 2, 2, 4)])
def test_gmres_iterates_match_the_oracle(shape, ndim, order, levels, steps):
    p, mask = _problem(shape, 41)
    say("gmres steps", shape, order, levels, steps)
    x, info = tikhonov_gmres(torch.from_numpy(p).cuda(), torch.from_numpy(mask).cuda(), ndim, order, levels, 1.0, 0.1,
                             iters=steps, restart=steps, rtol=0.0)
    assert info["iterations"] == steps
    for b in range(shape[0]):
        ref = oracle.tikhonov_gmres(p[b].astype(np.float64), mask[b].astype(np.float64), order, levels, 1.0, 0.1, steps)
        assert rel_l2(x[b].cpu().numpy(), ref) <= GMRES_TOL, b


@pytest.mark.parametrize("rtol", [0.3, 1e-2, 1e-4])
def test_gmres_stops_at_the_first_step_below_rtol(rtol):
    """The steps enqueued past the last needed one are not counted and do not enter x."""
    p, mask = _problem((2, 64, 96), 43)
    pt, mt = torch.from_numpy(p).cuda(), torch.from_numpy(mask).cuda()
    say("gmres rtol", rtol)

    def solve(iters, tol):
        return tikhonov_gmres(pt, mt, 2, 4, 4, 1.0, 0.1, iters=iters, restart=30, rtol=tol)

    x, info = solve(30, rtol)
    it = info["iterations"]
    assert 1 <= it < 30
    # the estimate is the true residual up to FP32 (1e-6 relative to ||b||)
    assert float(info["rel_residual"].max()) <= rtol + 1e-5
    _, before = solve(it - 1, 0.0)
    assert float(before["rel_residual"].max()) > rtol - 1e-5
    capped, cinfo = solve(it, rtol)
    assert cinfo["iterations"] == it and torch.equal(capped, x)


def test_gmres_without_steps():
    p, mask = _problem((2, 32, 32), 47)
    say("gmres without steps")
    for kw in (dict(iters=0, rtol=1e-6), dict(iters=5, rtol=1.0)):
        x, info = tikhonov_gmres(torch.from_numpy(p).cuda(), torch.from_numpy(mask).cuda(), 2, 3, 3, 1.0, 0.1, **kw)
        assert info["iterations"] == 0 and float(x.abs().max()) == 0.0
        assert rel_l2(info["rel_residual"].numpy(), np.ones(2)) <= 1e-6
