"""A walk pass gives the same outputs whatever its launch: workgroups of 256,
512 and 1024 threads, one entry range or many per workgroup, decisions kept in
LDS or, when the frontier is far larger than the launch was sized for, in
memory.  A tree that last walked a smaller set launches small grids into buffers
that still hold the large walk.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


def _walk(tree, theta):
    tree.walk(theta)
    return tree.lists()


# frontiers of the smaller walk: below 1024 entries (all in one launch), some
# thousands, and about a quarter of the large one
@pytest.mark.parametrize("n_small", [500, 5000, 20000, 80000])
@pytest.mark.parametrize("n", [100000, 400000])
def test_grids_agree(n, n_small):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = (torch.from_numpy(a).to(dev) for a in g.plummer(n, 23))
    small = slice(0, n_small)
    ctx = api.Context(0)
    tree = api.Tree(ctx, pos, mass, n_leaf=8)
    first = _walk(tree, 0.5)
    tree.rebuild(pos[small].contiguous(), mass[small].contiguous())
    few = _walk(tree, 0.5)
    assert len(few[0]) + len(few[1]) < len(first[0]) + len(first[1])
    tree.rebuild(pos, mass)
    again = _walk(tree, 0.5)
    np.testing.assert_array_equal(first[0], again[0])
    np.testing.assert_array_equal(first[1], again[1])
    tree.rebuild(pos[small].contiguous(), mass[small].contiguous())
    back = _walk(tree, 0.5)
    np.testing.assert_array_equal(few[0], back[0])
    np.testing.assert_array_equal(few[1], back[1])
    tree.close()
    ctx.close()
