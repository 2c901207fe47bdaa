"""A first walk without room for its estimate: the passes are sized on the host,
and the lists and forces are those of the walk with the estimate.  Whatever the
budget, a larger one never refuses what a smaller one took.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import _lib
from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


# sized: the least budget has no room for the estimate (many small leaves)
@pytest.mark.parametrize("n,n_leaf,theta,sized", [(20000, 8, 0.4, True), (4000, 4, 0.4, True), (30000, 32, 0.35, False),
                                                  (200000, 64, 0.4, False)])
def test_budgets(n, n_leaf, theta, sized):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = (torch.from_numpy(a).to(dev) for a in g.uniform_ball(n, 7 + n))
    kw = dict(p=6, theta=theta, variant="conserving")

    def solve(budget):
        """Node count, bytes of the tree, lists (None: refused), forces (None: refused)."""
        ctx = api.Context(0, budget_bytes=budget)
        nodes = base = lists = f = tree = None
        try:
            tree = api.Tree(ctx, pos, mass, n_leaf=n_leaf)
            nodes, base = tree.info()["nodes"], ctx.bytes_in_use()
            tree.walk(theta)
            lists = tree.lists()
            f = tree.evaluate(**kw).cpu().numpy()
        except _lib.TfmmError as e:
            assert e.status == _lib.ENOMEM
        if tree is not None:
            tree.close()
        ctx.close()
        return nodes, base, lists, f

    nodes, base, lists, f = solve(0)
    budget = base // 2
    while True:  # the least budget that admits the walk
        budget += budget // 16
        got = solve(budget)
        if got[2] is not None:
            break
    # the estimate's far pairs alone, which a budget has to hold twice over
    assert not sized or budget / 2 < base + 8 * nodes * min(1.65 * (1 + 2 / theta) ** 3, 400.0)
    solved = False
    for k in range(30):
        np.testing.assert_array_equal(got[2][0], lists[0])
        np.testing.assert_array_equal(got[2][1], lists[1])
        assert got[3] is not None or not solved, (k, budget)
        if got[3] is not None:
            solved = True
            np.testing.assert_array_equal(got[3], f)
        budget += budget // 8
        got = solve(budget)
        assert got[2] is not None, (k, budget)
    assert solved
