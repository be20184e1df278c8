"""A box of a batch against the same box alone.  With a named tile every output agrees bit for bit.  Left to the library, a
batch may take the marching kernels and the box alone the kernel of one node per thread: FP32 fields with fixed points
agree bit for bit all the same; velocities at points are sums of 64 products in another order (64 roundings a
step), and the fields of moment storage, whose gathered sums are taken in another order, agree to 32 roundings a step."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402

EPS = 2.0 ** -24
SHAPE, NBOXES, PER_BOX, STEPS = (24, 24, 24), 300, 2, 9


def _run(storage, boxes, tile, kind):
    """The boxes named, with the points, forces and initial flow that they have in the batch."""
    n = len(boxes) * PER_BOX
    lat = lbm.Lattice(SHAPE, storage, nboxes=len(boxes), tau=0.7, max_points=n, tile=tile)
    parts = [np.random.default_rng(100 + b) for b in boxes]
    rho = np.stack([1 + g.normal(scale=1e-3, size=SHAPE) for g in parts])
    u = np.stack([g.normal(scale=1e-3, size=(3,) + SHAPE) for g in parts])
    pos = np.concatenate([g.uniform(0, 24, (PER_BOX, 3)) for g in parts])
    frc = np.concatenate([g.normal(scale=1e-6, size=(PER_BOX, 3)) for g in parts])
    dev = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    lat.set_equilibrium(dev(rho), dev(u))
    vel = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    model = lbm.PointModel(inv_a=1.4, inv_aL=0.7) if kind == lbm.LB_COLLOIDS else lbm.PointModel()
    model.vel_out = vel
    p = dev(pos)
    lat.add_point_forces(p, dev(frc), dev(np.repeat(np.arange(len(boxes), dtype=np.int32), PER_BOX)), kind, model)
    lat.step(STEPS)
    r, v = lat.moments()
    lat.sync()
    lat.close()
    return r, v, vel, p


@pytest.mark.parametrize("storage", ["fp32", "mom32"])
@pytest.mark.parametrize("kind", [lbm.LB_FORCES_STATIC, lbm.LB_COLLOIDS])
def test_box_of_a_batch(storage, kind):
    moving = kind == lbm.LB_COLLOIDS
    plan = [lbm.lb_plan(lbm.make_params(SHAPE, storage, nboxes=k, max_points=k * PER_BOX), k * PER_BOX, 2 if moving else 1)
            for k in (NBOXES, 1)]
    assert (plan[0].march_planes > 0) == (storage == "mom32" or not moving) and plan[1].march_planes == 0
    for tile in ((32, 4, 2), None):
        batch = _run(storage, list(range(NBOXES)), tile, kind)
        for b in (0, 7, NBOXES - 1):
            one = _run(storage, [b], tile, kind)
            mine = [batch[0].reshape(NBOXES, -1)[b], batch[1].reshape(NBOXES, -1)[b], batch[2][b * PER_BOX:(b + 1) * PER_BOX],
                    batch[3][b * PER_BOX:(b + 1) * PER_BOX]]
            top = max(one[1].abs().max().item(), (one[0] - 1).abs().max().item())
            for k, (x, y) in enumerate(zip(mine, one)):
                y = y.reshape(x.shape)
                if tile or (storage == "fp32" and not moving and k < 2):
                    assert torch.equal(x, y), (tile, b, k)
                else:
                    assert (x - y).abs().max().item() <= STEPS * 64 * EPS * top * (STEPS if k == 3 else 1), (b, k)
