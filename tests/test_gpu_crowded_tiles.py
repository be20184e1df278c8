"""Tiles with no, few and many points, below and above what one staging round holds (51 records in FP32, 28 in
FP64), against the FP64 oracle: fields after a few steps and velocities at the points.  1e-10 of the largest
velocity in FP64, 1e-5 in FP32 and moment storage."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


@pytest.mark.parametrize("storage,bar", [("fp64", 1e-10), ("fp32", 1e-5), ("mom32", 1e-5)])
@pytest.mark.parametrize("tile,variant", [(None, 0), ((64, 2, 2), 128), ((16, 4, 4), 192), ((128, 2, 1), 130),
                                          ((32, 4, 2), 4)])
@pytest.mark.parametrize("npts", [3, 27, 30, 56, 120])
def test_crowded_tile(storage, bar, tile, variant, npts):
    shape = (9, 10, 70)
    g = np.random.default_rng(npts)
    ext = np.array(shape[::-1], dtype=np.float64)
    # half of the points in one cell across a tile corner, the rest anywhere
    pos = np.concatenate([np.array([63.6, 3.7, 3.6]) + g.uniform(0, 0.8, (npts - npts // 2, 3)),
                          g.uniform(0, 1, (npts // 2, 3)) * ext])
    frc = g.normal(scale=1e-6, size=(npts, 3))
    lat = lbm.Lattice(shape, storage, tau=0.8, max_points=npts, tile=tile, variant=variant)
    p = torch.tensor(pos, device="cuda")
    vel = torch.zeros_like(p)
    lat.add_point_forces(p, torch.tensor(frc, device="cuda"), None, lbm.LB_COLLOIDS,
                         lbm.PointModel(inv_a=2.0, inv_aL=0.7, vel_out=vel))
    lat.step(5)
    _, u = lat.moments()
    lat.sync()
    o = oracle.Box(shape, 0.8)
    o.sets = [oracle.ForceSet(pos.copy(), frc, kind="colloid", inv_a=2.0, inv_aL=0.7)]
    o.step(5)
    _, uo = o.moments()
    top = np.abs(uo).max()
    assert np.abs(u[0].cpu().numpy() - uo).max() <= bar * top
    assert np.abs(vel.cpu().numpy() - o.sets[0].U).max() <= bar * top
