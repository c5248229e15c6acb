"""GPU: 3-D non-periodic levels whose slices are so small that the split form would need 2^32 threads run as tiles, with
the bits that the same instances have in a small batch (split)."""
import pytest
import torch

import paper_2507_02401_amd as es
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fn", [es.sym_cov_apply, es.sym_cov_apply_transpose])
def test_batch_of_tiny_slices(fn):
    batch = (1 << 18) + 3
    say("sym tiny slices", batch)
    x = torch.randn((batch, 64, 4, 4), generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    got = fn(x, 3, 8, 2, 1.0)
    for k in (0, 1 << 17, batch - 4):
        assert torch.equal(got[k:k + 4], fn(x[k:k + 4].contiguous(), 3, 8, 2, 1.0))
