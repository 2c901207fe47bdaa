"""The FP32 near field of large trees, one wavefront per item, against the
workgroups of four or eight that small trees use: the same sums in the same
order.  The filler has 33000 or more leaves, each at least one item, more than
workgroups of several wavefronts are used for."""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


# leaves of one and of several 64-target chunks, every number of targets per lane
# (small leaves to full ones), items of one and of many source chunks
@pytest.mark.parametrize("n,n_leaf", [(65, 64), (257, 130), (1000, 5), (3001, 64), (4099, 200), (9973, 64), (2500, 130)])
@pytest.mark.parametrize("eps", [0.0, 1e-3])
def test_one_wavefront_equals_several_bitwise(n, n_leaf, eps):
    import torch

    from paper_2107_07166_amd import api

    pos, mass = g.plummer(n, 11 + n)
    fill, fmass = g.uniform_ball(33000 * n_leaf, 5)
    dev = torch.device("cuda:0")
    kw = dict(p=2, theta=0.5, eps=eps, variant="conserving", precision="mixed32")
    ctx = api.Context(0)
    tree = api.Tree(ctx, torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev), n_leaf=n_leaf)
    phi = torch.empty(n, dtype=torch.float64, device=dev)
    f = tree.evaluate(pot=phi, **kw).clone()
    assert tree.info()["leaves"] < 4096
    tree.close()
    mb = torch.from_numpy(np.concatenate([mass, fmass])).to(dev)
    tree = api.Tree(ctx, torch.from_numpy(np.concatenate([pos, fill])).to(dev), mb, n_leaf=n_leaf,
                    offsets=[0, n, n + len(fill)])
    phib = torch.empty_like(mb)
    fb = tree.evaluate(pot=phib, **kw)
    assert tree.info()["leaves"] > 32768
    assert torch.equal(f, fb[:n]) and torch.equal(phi, phib[:n])
    tree.close()
    ctx.close()
