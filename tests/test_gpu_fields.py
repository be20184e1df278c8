"""Set-up and read-out where the kernels change their way: velocity at points in plain order and slab by slab
(many points for the lattice), tile lists built by few and many blocks, reads that follow each other
without a step, equilibrium on rows of less and more than a wave.  Against the FP64 oracle: 1e-10
in FP64, 1e-5 in FP32 of the largest velocity."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


def _flow(shape, g):
    z, y, x = np.meshgrid(*[2 * np.pi * np.arange(n) / n for n in shape], indexing="ij")
    a = g.uniform(-1e-3, 1e-3, (3, 4))
    u = np.stack([a[c, 0] + a[c, 1] * np.sin(x + c) + a[c, 2] * np.cos(y) + a[c, 3] * np.sin(z - c) for c in range(3)])
    return 1.0 + 1e-3 * np.cos(x + y) * np.sin(z + 0.3), u


@pytest.mark.parametrize("storage,bar", [("fp64", 1e-10), ("fp32", 1e-5)])
@pytest.mark.parametrize("shape,npts,nforce", [((8, 6, 5), 3, 1), ((9, 10, 70), 3000, 40), ((20, 12, 16), 777, 1200),
                                               ((33, 7, 130), 5000, 5), ((70, 64, 50), 9000, 3)])
def test_equilibrium_and_velocity_at_points(storage, bar, shape, npts, nforce):
    g = np.random.default_rng(npts)
    ext = np.array(shape[::-1], dtype=np.float64)
    nb = 2
    flows = [_flow(shape, g) for _ in range(nb)]
    pos, frc = g.uniform(0, 1, (nforce, 3)) * ext, g.normal(scale=1e-6, size=(nforce, 3))
    box = g.integers(0, nb, nforce).astype(np.int32)
    at, abox = g.uniform(-0.5, 1.5, (npts, 3)) * ext, g.integers(0, nb, npts).astype(np.int32)
    dev = lambda v: torch.tensor(v, device="cuda")   # noqa: E731
    lat = lbm.Lattice(shape, storage, nboxes=nb, tau=0.7, max_points=nforce)
    lat.add_point_forces(dev(pos), dev(frc), dev(box))
    lat.set_equilibrium(dev(np.stack([f[0] for f in flows])), dev(np.stack([f[1] for f in flows])))
    first = lat.interp_velocity(dev(at), dev(abox))
    rho, u = lat.moments()
    again = lat.interp_velocity(dev(at), dev(abox))
    r, diag = lat.diagnostics()
    assert r == lbm.LB_OK and torch.equal(first, again)
    rho, u, got = rho.cpu().numpy(), u.cpu().numpy(), first.cpu().numpy()
    for b in range(nb):
        o = oracle.Box(shape, 0.7)
        o.df = oracle.equilibrium(flows[b][0], flows[b][1], 1.0)
        mine = box == b
        o.sets = [oracle.ForceSet(pos[mine], frc[mine])]
        ro, uo = o.moments()
        top = np.abs(uo).max()
        assert np.abs(u[b] - uo).max() <= bar * top
        assert np.abs(rho[b] - ro).max() <= bar
        assert np.abs(got[abox == b] - o.interp_velocity(at[abox == b])).max() <= bar * top
        assert abs(diag[b, 0] - (ro - 1.0).sum()) <= bar * np.abs(ro - 1.0).sum()
        assert np.abs(diag[b, 4:7] - frc[mine].sum(0)).max() <= bar * np.abs(frc[mine]).sum() + 1e-18
        assert abs(diag[b, 10] - np.sqrt((uo ** 2).sum(0)).max()) <= bar * top


def test_reads_follow_moved_points():
    """Positions of a set read at every call, rewritten between two reads: the lists follow."""
    shape, g = (24, 20, 40), np.random.default_rng(3)
    ext = np.array(shape[::-1], dtype=np.float64)
    pos = torch.tensor(g.uniform(0, 1, (50, 3)) * ext, device="cuda")
    frc = torch.tensor(g.normal(scale=1e-5, size=(50, 3)), device="cuda")
    lat = lbm.Lattice(shape, "fp64", tau=0.7, max_points=50)
    lat.add_point_forces(pos, frc, None, lbm.LB_COLLOIDS, lbm.PointModel(inv_a=2.0, inv_aL=0.7))
    for k in range(3):
        for _ in range(2):
            _, u = lat.moments()
            o = oracle.Box(shape, 0.7)
            o.sets = [oracle.ForceSet(pos.cpu().numpy(), frc.cpu().numpy())]
            _, uo = o.moments()
            assert np.abs(u[0].cpu().numpy() - uo).max() <= 1e-10 * np.abs(uo).max()
        pos.copy_(torch.tensor(g.uniform(0, 1, (50, 3)) * ext))
