"""The forest's particle sort: boxes gathered across sets, keys counted with
the set numbers, one or two passes over the set number.  Every set's keys and
order are those of the set alone, whose build takes another route.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


# one and two passes over the set number; sets of one particle, sets within one
# wavefront's 1024 particles and across several, sets beyond the small sort
@pytest.mark.parametrize("n_sets,largest", [(2, 3), (2, 20000), (17, 5000), (256, 700), (257, 700), (1500, 90)])
def test_sets_are_sorted_as_alone(n_sets, largest):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n_sets)
    counts = rng.integers(1, largest + 1, n_sets)
    counts[0], counts[-1] = largest, 1
    off = np.concatenate([[0], np.cumsum(counts)])
    pos, mass = g.plummer(int(off[-1]), 9)
    for k in range(n_sets):  # cubes of every scale and on both sides of zero; ties in some sets
        x = pos[off[k]:off[k + 1]]
        x *= 10.0 ** rng.integers(-3, 4)
        x += rng.normal(size=3)
        if k % 3 == 0:
            x[len(x) // 2:] = x[:len(x) - len(x) // 2]
    ctx = api.Context(0)
    d_pos, d_mass = torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev)
    tree = api.Tree(ctx, d_pos, d_mass, n_leaf=16, offsets=off)
    both = tree.export()
    tree.close()
    for k in sorted({0, 1, n_sets // 2, n_sets - 2, n_sets - 1}):
        a, b = off[k], off[k + 1]
        tree = api.Tree(ctx, d_pos[a:b].contiguous(), d_mass[a:b].contiguous(), n_leaf=16)
        alone = tree.export()
        tree.close()
        np.testing.assert_array_equal(both["keys"][a:b], alone["keys"])
        np.testing.assert_array_equal(both["order"][a:b] - a, alone["order"])
    for k in range(n_sets):
        keys, order = both["keys"][off[k]:off[k + 1]], both["order"][off[k]:off[k + 1]]
        np.testing.assert_array_equal(order - off[k], np.argsort(keys, kind="stable"))
    ctx.close()
