"""r_max where its routes change: a wavefront per node in sets of up to 16384
particles, else rows of 16 lanes, items of up to 4096 particles from 513 on, and
several items from 4097 on.  All are exact maxima, operation by operation.
"""
import numpy as np
import pytest

from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 65, 512, 4097, 16384, 16385, 60000])
@pytest.mark.parametrize("kind", ["plummer", "ties", "shell", "tiny"])
def test_rmax_is_exact(n, kind):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = g.plummer(n, 41)
    if kind == "ties":  # groups without extent, nodes of equal particles
        pos[n // 4:] = pos[np.arange(n - n // 4) % max(n // 8, 1)]
    elif kind == "shell":  # every group nearly as far as the farthest
        pos /= np.linalg.norm(pos, axis=1)[:, None]
    elif kind == "tiny":  # squares underflow
        pos *= 1e-162
    ctx = api.Context(0)
    tree = api.Tree(ctx, torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev), n_leaf=128)
    a = tree.export()
    tree.close()
    ctx.close()
    x = pos[a["order"]]
    for i in np.unique(np.concatenate([np.argsort(-a["count"])[:40], np.arange(0, len(a["count"]), 7)])):
        d = x[a["first"][i]:a["first"][i] + a["count"][i]] - a["com"][i]
        r2 = ((d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]).max()
        assert a["rmax"][i] == np.sqrt(r2), (i, a["count"][i])
