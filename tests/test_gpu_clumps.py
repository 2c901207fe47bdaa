"""Leaves of the deepest level whose particles coincide, far more of them than a
leaf or a near-field work item holds elsewhere: one list entry then stands for
many items' worth of sources.  The forces are the oracle's, and the same beside
a filler set that takes the lists down the sorted route.
"""
import numpy as np
import pytest

import oracle
import parity
from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


def _clumps(clumps, size, spread):
    """Clumps of coincident particles within a spread of single ones."""
    rng = np.random.default_rng(5)
    single, _ = g.uniform_ball(spread, 6)
    pos = np.concatenate([np.repeat(rng.uniform(-0.4, 0.4, (clumps, 3)), size, axis=0), single])
    return pos, rng.uniform(0.5, 1.5, len(pos)) / len(pos)


@pytest.mark.parametrize("clumps,size,spread,n_leaf", [(1, 5000, 40, 64), (1, 100000, 8, 4), (8, 20000, 12, 4)])
@pytest.mark.parametrize("precision", ["mixed32", "fp64"])
def test_coincident_clumps(clumps, size, spread, n_leaf, precision):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = _clumps(clumps, size, spread)
    n = len(pos)
    kw = dict(p=4, eps=1e-2, variant="conserving", precision=precision)
    ctx = api.Context(0)
    tree = api.Tree(ctx, torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev), n_leaf=n_leaf)
    f = tree.evaluate(theta=0.5, **kw).cpu().numpy()
    assert tree.info()["max_level"] == 21
    tree.close()
    # two particles of every clump and all single ones
    some = np.concatenate([np.arange(clumps) * size, np.arange(clumps) * size + size - 1, np.arange(n - spread, n)])
    ref = oracle.Tree(pos, mass, n_leaf=n_leaf, theta=0.5).forces(4, 1e-2, "conserving", targets=some)
    parity.gate(f[some], ref, precision, f"{clumps} clumps of {size}")
    if clumps > 1:
        fill, fmass = g.uniform_ball(1200000, 7)
        both = torch.from_numpy(np.concatenate([pos, fill])).to(dev)
        mb = torch.from_numpy(np.concatenate([mass, fmass])).to(dev)
        tree = api.Tree(ctx, both, mb, n_leaf=n_leaf, offsets=[0, n, n + len(fill)])
        assert tree.info()["nodes"] > 1 << 19
        fb = tree.evaluate(theta=0.5, **kw)[:n].cpu().numpy()
        np.testing.assert_array_equal(f, fb)
        tree.close()
    ctx.close()
