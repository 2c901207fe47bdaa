"""The walk's launches: small passes together in one workgroup, larger passes
in two launches each, and host-sized passes when the room runs out.  Whatever
the mixture, the pairs come out in the same order, so the lists of every route
have to be equal element by element (the pair sets themselves are compared with
the oracle's elsewhere).
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


def _walk(tree, theta):
    tree.walk(theta)
    return tree.lists()


def _same(a, b):
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


# one leaf; frontiers that stay in one workgroup, that leave it, and that come
# back with more passes than the walk before had
@pytest.mark.parametrize("n,n_leaf,theta", [(3, 64, 0.5), (2048, 64, 0.5), (3000, 4, 0.8), (30000, 16, 0.6),
                                            (200000, 64, 0.4)])
def test_routes_agree(n, n_leaf, theta):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = (torch.from_numpy(a).to(dev) for a in g.plummer(n, 7 + n))
    ctx = api.Context(0)
    tree = api.Tree(ctx, pos, mass, n_leaf=n_leaf)
    first = _walk(tree, theta)       # estimated room
    _same(first, _walk(tree, theta))  # sized from the walk before
    info = tree.info()
    held = ctx.bytes_held()
    # a tree that last walked a smaller set has too few launches and too little room
    small = api.Tree(ctx, pos[:max(n // 10, 1)].contiguous(), mass[:max(n // 10, 1)].contiguous(), n_leaf=n_leaf)
    small.walk(0.9)
    small.rebuild(pos, mass)
    _same(first, _walk(small, theta))
    small.close()
    tree.close()
    ctx.close()
    # a budget without room for the estimate: host-sized passes
    tight = api.Context(0, budget_bytes=max(held, 1 << 20))
    tree = api.Tree(tight, pos, mass, n_leaf=n_leaf)
    tight.set_budget(tight.bytes_held() + 16 * (info["far_pairs"] + info["near_pairs"]) * 4 + (8 << 20))
    _same(first, _walk(tree, theta))
    tree.close()
    tight.close()


# more roots than one workgroup's passes take, and more than fit its LDS
@pytest.mark.parametrize("n_sets", [1, 1025, 2500])
def test_many_roots(n_sets):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    per = 40
    pos, mass = (torch.from_numpy(a).to(dev) for a in g.uniform_ball(per * n_sets, 3))
    ctx = api.Context(0)
    off = np.arange(n_sets + 1) * per
    tree = api.Tree(ctx, pos, mass, n_leaf=8, offsets=off)
    first = _walk(tree, 0.5)
    _same(first, _walk(tree, 0.5))
    # every set's pairs are its own tree's: the set of a pair follows from its nodes' particles
    d = tree.export()
    sets = d["first"] // per
    for pairs in first:
        np.testing.assert_array_equal(sets[pairs[:, 0]], sets[pairs[:, 1]])
    k = n_sets // 2
    alone = api.Tree(ctx, pos[k * per:(k + 1) * per].contiguous(), mass[k * per:(k + 1) * per].contiguous(), n_leaf=8)
    af, an = _walk(alone, 0.5)
    assert int((sets[first[0][:, 0]] == k).sum()) == len(af)
    assert int((sets[first[1][:, 0]] == k).sum()) == len(an)
    alone.close()
    tree.close()
    ctx.close()
