"""GPU: 3-D low-pass analysis levels that run as planes and an axis-1 pass give the bits of the one-launch
tiles (ESWAVE_STREAMED=0), for every filter length that splits, on sides that leave partial tiles, partial
line groups and unaligned rows, in batches, through workspaces on dirty memory, and in a plan."""
import pytest
import torch

import paper_2507_02401_amd as es
from tests.gpu_util import env, say

pytestmark = pytest.mark.gpu

CASES = [  # shape, batch, order, levels
    ((96, 96, 96), 1, 8, 3),       # whole tiles, two levels below
    ((128, 64, 32), 26, 8, 3),     # the second level splits too; rows shorter than the window
    ((92, 100, 92), 1, 8, 2),      # partial tiles, lines cut off inside a 16-byte group (46 = 11 * 4 + 2)
    ((100, 36, 236), 1, 7, 2),
    ((20, 420, 100), 1, 6, 2),     # window longer than axis 0
    ((4, 448, 452), 1, 8, 2),      # 2 outputs along axis 0
    ((64, 128, 200), 1, 5, 3),
    ((176, 200, 184), 1, 4, 3),
]


def _names(shape, batch, order, levels):
    import ctypes

    from paper_2507_02401_amd import _lib
    lib, out, buf = _lib.load(), [], ctypes.create_string_buffer(128)
    while lib.es_schedule_describe(es.OP_COV, len(shape), _lib.shape_arg(shape), batch, order, levels, len(out), buf, 128, None,
                                   None) == 0:
        out.append(buf.value.decode())
    return out


@pytest.mark.parametrize("shape,batch,order,levels", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_split_levels_give_the_tiles_bits(shape, batch, order, levels):
    say("lp split", shape, batch, order, levels)
    assert any(n.startswith("lp_down_p") for n in _names(shape, batch, order, levels))
    x = torch.randn((batch,) + shape, generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    for fn in (es.matern_cov_apply, es.matern_sample):
        with env(ESWAVE_STREAMED="0"):
            ref = fn(x, 3, order, levels, 1.0)
        torch.full((4 * x.numel(),), float("nan"), device="cuda")  # dirty memory for the next allocations
        got = fn(x, 3, order, levels, 1.0)
        assert torch.equal(got, ref)


def test_split_levels_in_a_plan():
    descs = [((96, 96, 96), 8, 3, 1.0), ((48, 64, 64), 8, 3, 1.0), ((64, 64, 64), 8, 2, 0.5), ((64, 96), 8, 3, 1.0)]
    xs = [torch.randn(d[0], generator=torch.Generator("cuda").manual_seed(k), device="cuda") for k, d in enumerate(descs)]
    plan = es.RaggedPlan(descs, es.OP_COV)
    with env(ESWAVE_STREAMED="0"):
        refs = [es.matern_cov_apply(x[None], x.ndim, d[1], d[2], d[3])[0] for x, d in zip(xs, descs)]
    for graph in (False, True, True):
        for y, ref in zip(plan(xs, graph=graph), refs):
            assert torch.equal(y, ref)
    plan.close()
