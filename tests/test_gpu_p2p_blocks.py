"""The near field run by workgroups of one, four or eight wavefronts per item.

A set solved alone has few work items (eight or four wavefronts each); inside
a forest with a large filler set the same leaves are served by one wavefront
each.  The chunk sums are added in the same order, so the forces and the
potential have to agree bit for bit.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


# sizes around one chunk of 256 sources, odd leaves, leaves of more than one
# 64-target chunk, and more than eight chunks per item
@pytest.mark.parametrize("n,n_leaf", [(1, 64), (65, 64), (257, 130), (1000, 5), (3001, 64), (4099, 200), (9973, 64)])
@pytest.mark.parametrize("precision", ["mixed32", "fp64"])
@pytest.mark.parametrize("eps", [0.0, 1e-3])
def test_block_sizes_agree_bitwise(n, n_leaf, precision, eps):
    import torch

    from paper_2107_07166_amd import api

    pos, mass = g.plummer(n, 11 + n)
    fill, fmass = g.uniform_ball(20000 * min(n_leaf, 16), 5)
    ctx = api.Context(0)
    dev = torch.device("cuda:0")
    kw = dict(p=2, theta=0.5, eps=eps, variant="conserving", precision=precision)
    pa, ma = torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev)
    tree = api.Tree(ctx, pa, ma, n_leaf=n_leaf)
    phi = torch.empty_like(ma)
    f = tree.evaluate(pot=phi, **kw).clone()
    f0 = tree.evaluate(**kw).cpu().numpy()
    tree.close()
    both = torch.from_numpy(np.concatenate([pos, fill])).to(dev)
    mb = torch.from_numpy(np.concatenate([mass, fmass])).to(dev)
    tree = api.Tree(ctx, both, mb, n_leaf=n_leaf, offsets=[0, n, n + len(fill)])
    phib = torch.empty_like(mb)
    fb = tree.evaluate(pot=phib, **kw)
    assert tree.info()["leaves"] > 8192 or n_leaf > 64  # the filler's leaves: one wavefront per item
    np.testing.assert_array_equal(f.cpu().numpy(), fb[:n].cpu().numpy())
    np.testing.assert_array_equal(phi.cpu().numpy(), phib[:n].cpu().numpy())
    np.testing.assert_array_equal(f0, f.cpu().numpy())
    tree.close()
    ctx.close()
