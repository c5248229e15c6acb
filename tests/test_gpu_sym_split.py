"""GPU: 3-D non-periodic analysis levels that run split (the 2-D level over the slices, then axis 0),
at the sizes where the split starts, where its scratch does not fit and on odd sides."""
import numpy as np
import pytest
import torch

import paper_2507_02401_amd as es
from oracle import symdwt
from tests.gpu_util import TOL, rel_l2, say

pytestmark = pytest.mark.gpu
DEV = "cuda"


# 14 and 16 taps split at every size: sides shorter than a chunk, than the filter (scratch too small:
# the 3-D tile runs), unaligned rows, more than one 256-thread block per slice
@pytest.mark.parametrize("shape,batch,order,levels", [
    ((3, 4, 5), 2, 8, 3), ((15, 15, 15), 1, 8, 2), ((17, 23, 31), 3, 7, 3), ((8, 40, 40), 1, 8, 3),
    ((41, 19, 26), 2, 8, 4), ((5, 100, 129), 1, 7, 2), ((64, 24, 24), 1, 8, 2)])
def test_split_levels_match_the_oracle(shape, batch, order, levels):
    x = np.random.default_rng(sum(shape) + order).standard_normal((batch,) + shape).astype(np.float32)
    say("sym split", shape, batch, order, levels)
    xt = torch.from_numpy(x).to(DEV)
    fwd = es.sym_cov_apply(xt, 3, order, levels, 1.0).cpu().numpy()
    tr = es.sym_cov_apply_transpose(xt, 3, order, levels, 1.0).cpu().numpy()
    for b in range(batch):
        x64 = x[b].astype(np.float64)
        assert rel_l2(fwd[b], symdwt.sym_cov_apply(x64, order, levels, 1.0)) < TOL
        assert rel_l2(tr[b], symdwt.sym_cov_apply_transpose(x64, order, levels, 1.0)) < TOL


@pytest.mark.parametrize("order,batch", [(3, 17), (4, 9), (5, 5), (6, 3)])
def test_split_and_tile_give_the_same_bits(order, batch):
    """Filters of 6 to 12 taps split from 2^(25 - order) samples of a call on: the batch runs split, its
    instances alone run the 3-D tile, and each sums its taps in the same order."""
    shape = (61, 66, 67)
    n = int(np.prod(shape))
    assert n < 1 << (25 - order) <= batch * n
    say("sym split bits", order, batch)
    x = torch.from_numpy(np.random.default_rng(order).standard_normal((batch,) + shape).astype(np.float32)).to(DEV)
    for fn in (es.sym_cov_apply, es.sym_cov_apply_transpose):
        whole = fn(x, 3, order, 3, 1.0)
        for b in (0, batch - 1):
            assert torch.equal(whole[b], fn(x[b].contiguous(), 3, order, 3, 1.0))
