"""The downward pass from order 5: one launch per level in large trees, one
launch carrying every leaf's expansion down from the root in small ones.  The
shifts are the same in the same order, so a small set solved alone and the same
set in a forest with a large filler agree bit for bit.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,variant,precision", [(5, "conserving", "mixed32"), (5, "standard", "fp64"),
                                                 (6, "conserving", "fp64"), (6, "standard", "mixed32"),
                                                 (8, "conserving", "mixed32"), (8, "standard", "mixed32")])
# a single leaf (no far list at all), shallow and deep trees
@pytest.mark.parametrize("n,n_leaf", [(4, 4), (700, 4), (6001, 4)])
def test_chain_equals_levels_bitwise(p, variant, precision, n, n_leaf):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = g.plummer(n, 21)
    fill, fmass = g.uniform_ball(250000, 22)
    ctx = api.Context(0)
    kw = dict(p=p, theta=0.8, eps=1e-3, variant=variant, precision=precision)
    tree = api.Tree(ctx, torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev), n_leaf=n_leaf)
    f = tree.evaluate(**kw).cpu().numpy()
    tree.close()
    tree = api.Tree(ctx, torch.from_numpy(np.concatenate([pos, fill])).to(dev),
                    torch.from_numpy(np.concatenate([mass, fmass])).to(dev), n_leaf=n_leaf,
                    offsets=[0, n, n + len(fill)])
    assert tree.info()["leaves"] > 65536  # the level launches, also with one thread per leaf
    fb = tree.evaluate(**kw)[:n].cpu().numpy()
    tree.close()
    ctx.close()
    np.testing.assert_array_equal(f, fb)
