"""lb_set_equilibrium over rows of all widths (several to a wave, one, parts of one) and ends of boxes inside a wave: the
moments of the state it sets are the density and velocity it was given (moment storage takes the equilibrium as the state
after a collision: its moments are those of the equilibrium one propagation later), to the rounding of their sums: 91
pieces in moment storage, 19 populations otherwise, of at most the density's deviation plus three times the velocity."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402

C = [c for c in np.ndindex(3, 3, 3) if sum(abs(v - 1) for v in c) < 3]          # (z, y, x) + 1
W = {0: 1 / 3, 1: 1 / 18, 2: 1 / 36}


def _propagated(rho, u):
    """density and velocity of the equilibrium of (rho, u) after one propagation"""
    r, j = torch.zeros_like(rho), torch.zeros_like(u)
    for c in C:
        z, y, x = (v - 1 for v in c)
        cu = x * u[:, 0] + y * u[:, 1] + z * u[:, 2]
        f = W[abs(x) + abs(y) + abs(z)] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(1))
        f = torch.roll(f, (z, y, x), (1, 2, 3))
        r += f
        j += torch.stack([x * f, y * f, z * f], 1)
    return r, j / r[:, None]


EPS = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24, "mom32": 2.0 ** -24, "fp16": 2.0 ** -11}


@pytest.mark.parametrize("shape,nboxes", [
    ((4, 4, 4), 7), ((13, 30, 5), 3), ((9, 9, 9), 5), ((6, 5, 16), 3), ((5, 7, 31), 2), ((4, 4, 32), 3), ((6, 5, 33), 2),
    ((5, 4, 64), 2), ((7, 6, 65), 2), ((4, 5, 130), 1), ((4, 4, 257), 2),
])
@pytest.mark.parametrize("storage", ["fp32", "fp64", "mom32", "fp16"])
def test_moments_give_the_field_back(shape, nboxes, storage):
    g = np.random.default_rng(3)
    rho = torch.tensor(1 + g.uniform(-1e-3, 1e-3, (nboxes,) + shape), device="cuda")
    u = torch.tensor(g.uniform(-1e-3, 1e-3, (nboxes, 3) + shape), device="cuda")
    lat = lbm.Lattice(shape, storage, nboxes=nboxes, tau=0.7, fp16_exponent=16 if storage == "fp16" else 0)
    lat.set_equilibrium(rho, u)
    r, v = lat.moments()
    lat.sync()
    if storage == "mom32":
        rho, u = _propagated(rho, u)
    tol = (91 if storage == "mom32" else 19) * EPS[storage] * 4e-3 + 4 * 2.0 ** -53
    assert (r - rho).abs().max().item() <= tol
    assert (v - u).abs().max().item() <= 2 * tol
