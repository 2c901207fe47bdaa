"""A rebuild that fails leaves no tree behind: neither the old particles' lists
nor the new ones' sizes serve another call, and the next rebuild is as good as
a fresh tree."""
import numpy as np
import pytest

from paper_2107_07166_amd import _lib
from paper_2107_07166_amd import generators as g

pytestmark = pytest.mark.gpu

KW = dict(p=3, theta=0.6)


def _refused(call):
    with pytest.raises(_lib.TfmmError) as e:
        call()
    assert e.value.status == _lib.ESTATE


# the refused set smaller than, as large as and larger than the one before, on
# both routes of the build
# (memory: the larger ones)
SIZES = [(3000, 900), (3000, 3000), (3000, 40000), (30000, 30000), (30000, 200000)]
CASES = [(how, *s) for how in ("nan", "forest", "memory") for s in SIZES if how != "memory" or s[1] > s[0]]


@pytest.mark.parametrize("how,n,n_bad", CASES)
def test_nothing_is_left_of_a_refused_rebuild(how, n, n_bad):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    pos, mass = (torch.from_numpy(a).to(dev) for a in g.plummer(n, 4))
    bad, bmass = (torch.from_numpy(a).to(dev) for a in g.uniform_ball(n_bad, 5))
    offsets = [0, n_bad // 3, n_bad] if how == "forest" else None
    ctx = api.Context(0)
    tree = api.Tree(ctx, pos, mass)
    f = tree.evaluate(**KW).clone()
    status = _lib.EINVAL
    if how == "memory":
        ctx.trim()
        ctx.set_budget(ctx.bytes_held())
        status = _lib.ENOMEM
    else:
        bad[n_bad // 2, 1] = float("nan")
    with pytest.raises(_lib.TfmmError) as e:
        tree.rebuild(bad, bmass, offsets=offsets)
    assert e.value.status == status
    ctx.set_budget(0)
    out = torch.full_like(pos, 7.0)
    _refused(lambda: tree.evaluate(out=out, **KW))
    _refused(lambda: tree.evaluate_forest([0.6], p=3))
    _refused(lambda: tree.walk(0.6))
    _refused(tree.export)
    _refused(tree.lists)
    assert bool((out == 7.0).all())
    assert tree.info()["n"] == n
    tree.rebuild(pos, mass)
    assert torch.equal(f, tree.evaluate(**KW))
    tree.close()
    ctx.close()


def test_a_session_goes_on_after_a_refused_step():
    """Steps of a session need no build from before: one whose positions were
    spoilt and put right again goes on as if nothing had been."""
    import torch

    from paper_2107_07166_amd import api, session

    dev = torch.device("cuda:0")
    pos, mass = g.plummer(5000, 8)
    vel = np.random.default_rng(1).normal(0, 0.3, pos.shape)
    ctx = api.Context(0)
    ses = [session.Session(ctx, *(torch.from_numpy(a.copy()).to(dev) for a in (pos, vel, mass)), **KW) for _ in range(2)]
    for s in ses:
        s.step(1e-3, 1)
    keep = {k: getattr(ses[0], k).clone() for k in ("pos", "vel", "force")}
    ses[0].pos[17, 2] = float("inf")
    with pytest.raises(_lib.TfmmError):
        ses[0].step(1e-3, 1)
    for k, v in keep.items():
        getattr(ses[0], k).copy_(v)
    for s in ses:
        s.step(1e-3, 2)
    for k in keep:
        assert torch.equal(getattr(ses[0], k), getattr(ses[1], k)), k
    for s in ses:
        s.close()
    ctx.close()
