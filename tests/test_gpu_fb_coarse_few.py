"""GPU: full-bank coarse launches of at most one 3-D block per CU run another size of the kernel than larger batches
do: the same bits, on both sides of the limit and of the rule's filter lengths."""
import numpy as np
import pytest
import torch

import paper_2507_02401_amd as es
from tests.gpu_util import ORACLE_OPS, TOL, rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [1, 2, 4, 6, 7])
@pytest.mark.parametrize("shape", [(16, 16, 16), (8, 16, 24), (16, 16, 12), (8, 8, 8)], ids=str)
def test_batches_equal_their_instances(shape, order):
    x = torch.randn((257,) + shape, generator=torch.Generator("cuda").manual_seed(order), device="cuda")
    say("full-bank coarse, few blocks", shape, order)
    for fn, ref in zip((es.es_adjoint, es.es_apply), ORACLE_OPS):
        many = fn(x, 3, order, 2, 1.0)
        assert torch.equal(many[:256], fn(x[:256].contiguous(), 3, order, 2, 1.0))
        one = fn(x[256].contiguous(), 3, order, 2, 1.0)
        assert torch.equal(many[256], one)
        assert rel_l2(one.cpu().numpy(), ref(x[256].cpu().numpy().astype(np.float64), order, 2, 1.0)) < TOL
