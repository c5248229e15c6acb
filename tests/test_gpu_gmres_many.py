"""GPU: GMRES on so many small instances that a launch of 1024 threads an instance would hold 2^32 threads; every
instance has the bits that it has in a small batch."""
import pytest
import torch

from paper_2507_02401_amd import solver
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def test_four_million_instances():
    batch = (1 << 22) + 5
    say("gmres many", batch)
    gen = torch.Generator("cuda").manual_seed(4)
    p = torch.randn((batch, 2, 2), generator=gen, device="cuda")
    mask = (torch.rand((batch, 2, 2), generator=gen, device="cuda") < 0.7).float()
    got, info = solver.tikhonov_gmres(mask * p, mask, 2, 1, 1, 1.0, 0.05, iters=2, restart=2, rtol=0.0)
    assert info["iterations"] == 2
    for k in (0, 1 << 21, batch - 8):
        part = slice(k, k + 8)
        ref, _ = solver.tikhonov_gmres((mask * p)[part].contiguous(), mask[part].contiguous(), 2, 1, 1, 1.0, 0.05, iters=2,
                                       restart=2, rtol=0.0)
        assert torch.equal(got[part], ref)
