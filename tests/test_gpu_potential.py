"""The far-field potential shares the standard forces' locals, and has locals
of its own beside the other variants' forces.  Both are the standard expansion
of the same order, and asking for the potential leaves the forces alone.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["mixed32", "fp64"])
@pytest.mark.parametrize("p,n", [(1, 500), (2, 3000), (4, 9001), (5, 9001), (8, 3000)])
def test_shared_and_own_locals_agree(p, n, precision):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = (torch.from_numpy(a).to(dev) for a in g.plummer(n, 17 + p))
    ctx = api.Context(0)
    tree = api.Tree(ctx, pos, mass, n_leaf=16)
    phi = {}
    for variant in ("standard", "conserving") + (("conserving_r2",) if p == 1 else ()):
        kw = dict(p=p, theta=0.6, variant=variant, precision=precision)
        alone = tree.evaluate(**kw).clone()
        phi[variant] = torch.empty(n, dtype=torch.float64, device=dev)
        assert torch.equal(tree.evaluate(pot=phi[variant], **kw), alone), variant
    tree.close()
    ctx.close()
    ref = phi.pop("standard").cpu().numpy()
    for variant, v in phi.items():
        # the same FP32 or FP64 locals, carried down in FP64 (order 5 and up in another order)
        np.testing.assert_allclose(v.cpu().numpy(), ref, rtol=1e-13, err_msg=variant)
