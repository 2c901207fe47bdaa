"""The list building's routes: one or several partition tiles, few or many
nodes (items in one launch, one-word or two-word entries, bucket or sorted
lists).  A set's lists, and with them its forces in every bit, are the same
alone and beside filler sets that take the tree to either side of each limit.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu

N_LEAF, THETA = 4, 0.2


def _solve(ctx, pos, mass, offsets):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    tree = api.Tree(ctx, torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev), n_leaf=N_LEAF,
                    offsets=offsets if len(offsets) > 2 else None)
    f = tree.evaluate(p=3, theta=THETA).cpu().numpy()
    info = tree.info()
    tree.close()
    return f, info


# n = 12: one tile; 5000: several tiles, lists of several items
@pytest.mark.parametrize("n", [12, 5000])
@pytest.mark.parametrize("nodes", [4096, 4097, 65536, 65537, 1 << 19, (1 << 19) + 1])
def test_routes_agree(n, nodes):
    from paper_2107_07166_amd import api

    pos, mass = g.plummer(n, 3 + n)
    fill, fmass = g.plummer(400, 5)
    ctx = api.Context(0)
    alone, info = _solve(ctx, pos, mass, [0, n])
    per_set = _solve(ctx, fill, fmass, [0, 400])[1]["nodes"]
    # filler sets, then sets of one particle (one node each) up to the count
    m, ones = divmod(nodes - info["nodes"], per_set)
    counts = [n] + [400] * m + [1] * ones
    offsets = np.concatenate([[0], np.cumsum(counts)])
    f, both = _solve(ctx, np.concatenate([pos] + [fill] * m + [fill[:ones]]),
                     np.concatenate([mass] + [fmass] * m + [fmass[:ones]]), offsets)
    ctx.close()
    assert both["nodes"] == nodes
    np.testing.assert_array_equal(f[:n], alone)
    # every copy of the filler as well, whichever buckets it fell into
    copies = f[n:n + 400 * m].reshape(m, 400, -1)
    np.testing.assert_array_equal(copies, np.broadcast_to(copies[:1], copies.shape))
