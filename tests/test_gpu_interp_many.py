"""Velocity at more points than one launch takes (2 ** 23; in slab order, which this lattice takes with 64 slabs, 2 ** 24 are
2 ** 32 threads): the call gives what calls on parts of the points give, bit for bit, since a point's velocity does not
depend on the others."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


@pytest.mark.parametrize("n", [(1 << 23) + 1, (1 << 24) - 64, (1 << 24) + 5, 3 << 23])
def test_many_points(n):
    shape = (128, 128, 128)
    g = torch.Generator(device="cuda").manual_seed(4)
    lat = lbm.Lattice(shape, "fp32", tau=0.7, nboxes=2)
    rho = torch.ones((2,) + shape, dtype=torch.float64, device="cuda")
    u = 1e-3 * torch.randn((2, 3) + shape, dtype=torch.float64, device="cuda", generator=g)
    lat.set_equilibrium(rho, u)
    pos = 128 * torch.rand((n, 3), dtype=torch.float64, device="cuda", generator=g)
    box = torch.randint(0, 2, (n,), dtype=torch.int32, device="cuda", generator=g)
    whole = lat.interp_velocity(pos, box)
    lat.sync()
    for a in range(0, n, 1 << 22):
        part = lat.interp_velocity(pos[a:a + (1 << 22)], box[a:a + (1 << 22)])
        assert torch.equal(whole[a:a + (1 << 22)], part)
    assert whole.abs().max().item() > 1e-4


@pytest.mark.parametrize("shape,storage", [
    ((64, 64, 64), "fp64"), ((40, 96, 128), "fp64"), ((300, 30, 36), "fp64"), ((70, 64, 64), "fp32"),
])
def test_slabs_of_all_heights(shape, storage):
    """40 slabs of FP64 lattices with fewer than four planes a slab, 64 of others, against plain order (few points)."""
    n = 40000
    g = torch.Generator(device="cuda").manual_seed(5)
    lat = lbm.Lattice(shape, storage, tau=0.7)
    u = 1e-3 * torch.randn((1, 3) + shape, dtype=torch.float64, device="cuda", generator=g)
    lat.set_equilibrium(torch.ones((1,) + shape, dtype=torch.float64, device="cuda"), u)
    pos = 400 * torch.rand((n, 3), dtype=torch.float64, device="cuda", generator=g) - 50
    whole = lat.interp_velocity(pos)
    for a in range(0, n, 500):
        assert torch.equal(whole[a:a + 500], lat.interp_velocity(pos[a:a + 500]))
