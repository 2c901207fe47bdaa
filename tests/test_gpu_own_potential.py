"""The near field adds every particle's own term -m / eps to its potential and the
last kernel takes it away again, by the same operations: it leaves nothing
behind, however much larger than the rest it is.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _potential(pos, mass, per_set, eps, precision):
    import torch

    from paper_2107_07166_amd import api

    dev = torch.device("cuda:0")
    ctx = api.Context(0)
    pd, md = torch.from_numpy(pos).to(dev), torch.from_numpy(mass).to(dev)
    tree = api.Tree(ctx, pd, md, offsets=np.arange(0, len(mass) + 1, per_set))
    phi = torch.empty_like(md)
    tree.evaluate(p=2, theta=0.5, eps=eps, variant="standard", precision=precision, pot=phi)
    tree.close()
    ctx.close()
    return phi.cpu().numpy()


@pytest.mark.parametrize("eps", [1.0, 0.3, 1e-3, 1.7e-6, 1e-9])
@pytest.mark.parametrize("precision", ["mixed32", "fp64"])
def test_lone_particles_have_no_potential(eps, precision):
    rng = np.random.default_rng(3)
    n = 2000
    phi = _potential(rng.normal(size=(n, 3)), rng.uniform(1e-3, 1.0, n), 1, eps, precision)
    np.testing.assert_array_equal(phi, 0.0)


@pytest.mark.parametrize("eps", [1.0, 0.3, 1e-3, 1.7e-6, 1e-9])
def test_pairs_in_double_precision(eps):
    """Two particles at a distance: the partner's term, to the rounding of its
    sum with the own term (half a unit in the last place of the sum, and a few
    of the partner's)."""
    rng = np.random.default_rng(4)
    n = 2000
    pos, mass = rng.normal(size=(2 * n, 3)), rng.uniform(1e-3, 1.0, 2 * n)
    phi = _potential(pos, mass, 2, eps, "fp64")
    r2 = ((pos[0::2] - pos[1::2]) ** 2).sum(1)
    partner = np.stack([mass[1::2], mass[0::2]], 1).reshape(-1) / np.repeat(np.sqrt(r2 + eps * eps), 2)
    assert (np.abs(phi + partner) <= 0.5 * np.spacing(mass / eps + partner) + 1e-14 * partner).all()
