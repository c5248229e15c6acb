"""GPU: plans whose 2-D launches hold several filter lengths give the bits of the one-geometry calls: every
filter length in one plan, both coarse sizes, rows that take the vector and the scalar synthesis, every
tile variant, next to 3-D instances (their own launches)."""
import pytest
import torch

import paper_2507_02401_amd as es
from tests.gpu_util import env, say

pytestmark = pytest.mark.gpu

SHAPES = [(512, 512), (360, 600), (96, 200), (40, 72), (256, 1024), (72, 40)]
DESCS = [(SHAPES[k % len(SHAPES)], 1 + k % 8, 3, (0.5, 1.0, 2.0)[k % 3]) for k in range(24)] + [((64, 64, 64), 3, 3, 1.0)]


@pytest.mark.parametrize("op", ["OP_COV", "OP_SAMPLE"])
@pytest.mark.parametrize("variant", ["", "0", "1", "2"])
def test_mixed_launches_give_the_calls_bits(op, variant):
    say("ragged mixed", op, variant)
    gen = torch.Generator("cuda").manual_seed(5)
    xs = [torch.randn(d[0], generator=gen, device="cuda") for d in DESCS]
    fn = es.matern_cov_apply if op == "OP_COV" else es.matern_sample
    refs = [fn(x[None], x.ndim, d[1], d[2], d[3])[0] for x, d in zip(xs, DESCS)]
    with env(ESWAVE_FORCE_VARIANT=variant):
        plan = es.RaggedPlan(DESCS, getattr(es, op))
        assert plan.num_launches < 30  # one filter length per launch: more than 60
        for graph in (False, True, True):
            outs = plan(xs, graph=graph)
            torch.cuda.synchronize()
            for k, (y, ref) in enumerate(zip(outs, refs)):
                assert torch.equal(y, ref), (k, DESCS[k], graph)
        plan.close()
