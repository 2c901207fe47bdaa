"""Several leapfrog steps in one call, whose kicks between two force evaluations
are one launch, equal the same steps in calls of their own bit for bit."""
import numpy as np
import pytest

from paper_2107_07166_amd.generators import polytrope_binary

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 129, 1500])
@pytest.mark.parametrize("calls", [(4,), (1, 1, 1, 1), (3, 0, 1)])
def test_steps_in_one_call_or_many(n, calls):
    import torch

    from paper_2107_07166_amd import api
    from paper_2107_07166_amd.session import Session

    pos, mass, vel = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in polytrope_binary(n, 5))  # two of n
    ctx = api.Context(0)

    def run(parts):
        s = Session(ctx, pos, vel, mass, p=2, n_leaf=16)
        for k in parts:
            s.step(1e-3, k)
        return s.pos.clone(), s.vel.clone()

    (x, v), (x1, v1) = run(calls), run((2, 2))
    ctx.close()
    assert torch.equal(x, x1) and torch.equal(v, v1)
