"""The marching step kernels (two FP32 steps per launch, one step of moment storage) against the kernels of one node per
thread, on shapes whose default they are: planes taken whole (up to 256, 576 and 1024 nodes; list tiles 16, 32 and
64 nodes wide) and cut ones, ragged both ways, wrapped round a narrow box, with chunks that do not divide the height.

FP32: density and velocity fields agree bit for bit with a named tile, over every way of splitting a run into calls (pairs
of steps, single steps, graphs).  Velocities at points agree bit for bit between the splits, and with the named
tile to the rounding of their partial sums: 64 products, each to 2 ** -24, per step.
Moment storage: the gathered sums are taken in another order, 32 roundings a step."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402

EPS = 2.0 ** -24


def _points(shape, nboxes, n, seed=3, crowd=0):
    g = np.random.default_rng(seed)
    pos = g.uniform(0, 1, (n, 3)) * np.array(shape[::-1], dtype=np.float64)
    box = g.integers(0, nboxes, n).astype(np.int32)
    if crowd:                                   # all of these in the plane z = 2 of box 0
        pos[:crowd, 2] = 2.25
        box[:crowd] = 0
    return (torch.tensor(pos, device="cuda"), torch.tensor(g.normal(scale=1e-6, size=(n, 3)), device="cuda"),
            torch.tensor(box, device="cuda"))


def _run(shape, nboxes, storage, n, tile, split, crowd=0, kind=lbm.LB_FORCES_STATIC, flow=False, **kw):
    lat = lbm.Lattice(shape, storage, nboxes=nboxes, tau=np.linspace(0.6, 0.9, nboxes), max_points=n, tile=tile,
                      variant=64 if tile else 0, **kw)
    if flow:
        g = np.random.default_rng(6)
        lat.set_equilibrium(torch.tensor(1 + g.normal(scale=1e-3, size=(nboxes,) + shape), device="cuda"),
                            torch.tensor(g.normal(scale=1e-3, size=(nboxes, 3) + shape), device="cuda"))
    pos, frc, box = _points(shape, nboxes, n, crowd=crowd)
    vel = torch.zeros_like(pos)
    if n:
        model = lbm.PointModel(inv_a=1.4, inv_aL=0.7) if kind == lbm.LB_COLLOIDS else lbm.PointModel()
        model.vel_sum = vel
        lat.add_point_forces(pos, frc, box, kind, model)
    for s in split:
        lat.step(s)
    rho, u = lat.moments()
    lat.sync()
    lat.close()
    return rho, u, vel, pos


@pytest.mark.parametrize("shape,nboxes,n,crowd", [
    ((16, 16, 16), 700, 900, 0),
    ((13, 30, 9), 600, 500, 0),            # odd rows, list tiles of 16 nodes
    ((24, 24, 24), 300, 400, 70),          # more records in a plane than are staged at once
    ((32, 32, 32), 300, 300, 0),
    ((21, 20, 50), 200, 300, 70),          # list tiles of 64 nodes
    ((128, 128, 128), 1, 149, 60),
    ((160, 100, 190), 1, 120, 0),          # ragged cuts, a last chunk of its own height
    ((40, 72, 60), 40, 200, 0),            # cuts wider than the box
    ((128, 128, 128), 1, 0, 0),
])
def test_two_steps_per_launch(shape, nboxes, n, crowd):
    zn = n % 2 == 0
    a = _run(shape, nboxes, "fp32", n, (64, 4, 1), [11], crowd, flow=n == 0, zero_net_force=zn)
    first = None
    for split in ([11], [1] * 11, [2, 9], [3, 4, 4], [6, 5]):
        b = _run(shape, nboxes, "fp32", n, None, split, crowd, flow=n == 0, zero_net_force=zn)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), split
        if n:
            first = b[2] if first is None else first
            assert torch.equal(first, b[2]), split
            assert (a[2] - b[2]).abs().max().item() <= 11 * 64 * EPS * a[1].abs().max().item()


def test_sets_that_come_and_go():
    """A next-step set, points that move (single steps on other tiles) and a return to fixed ones."""
    shape, nboxes = (24, 24, 24), 300
    out = []
    for tile in ((64, 4, 1), None):
        lat = lbm.Lattice(shape, "fp32", nboxes=nboxes, tau=0.7, max_points=900, tile=tile, variant=64 if tile else 0)
        sets = [_points(shape, nboxes, 300, seed=s) for s in range(4)]
        lat.add_point_forces(*sets[0])
        lat.step(9)
        lat.add_point_forces(*sets[1], lbm.LB_FORCES_NEXT_STEP)
        lat.step(9)
        lat.add_point_forces(*sets[2], lbm.LB_COLLOIDS, lbm.PointModel(inv_a=1.4, inv_aL=0.7))
        lat.step(6)
        lat.clear_forces()
        lat.step(5)
        lat.add_point_forces(*sets[3])
        lat.step(8)
        lat.add_point_forces(*sets[0])       # the force density is laid out again
        lat.step(8)
        out.append(lat.moments() + (sets[2][0],))
        lat.sync()
        lat.close()
    (ra, ua, pa), (rb, ub, pb) = out
    # the moved points' positions carry their velocities' rounding, and the fields with them
    top = ua.abs().max().item()
    assert (pa - pb).abs().max().item() <= 6 * 64 * EPS * top
    assert (ua - ub).abs().max().item() <= 45 * 64 * EPS * top
    assert (ra - rb).abs().max().item() <= 45 * 64 * EPS * top


@pytest.mark.parametrize("shape,nboxes,n", [((24, 24, 24), 300, 200), ((128, 128, 128), 1, 100)])
def test_checkpoints(shape, nboxes, n):
    def make():
        lat = lbm.Lattice(shape, "fp32", nboxes=nboxes, tau=0.7, max_points=n)
        pos, frc, box = _points(shape, nboxes, n)
        lat.add_point_forces(pos, frc, box)
        return lat

    a, b = make(), make()
    a.step(7)
    buf = torch.empty(a.checkpoint_bytes() + 256, dtype=torch.uint8, device="cuda")
    a.checkpoint_save(buf)
    a.step(9)
    b.step(4)
    b.checkpoint_load(buf)
    b.step(9)
    _, ua = a.moments()
    _, ub = b.moments()
    a.sync()
    assert b.steps_taken() == 16 and torch.equal(ua, ub)
    # a context with moving points uses other tiles; it takes the same checkpoint
    c = lbm.Lattice(shape, "fp32", nboxes=nboxes, tau=0.7, max_points=n)
    c.add_point_forces(*_points(shape, nboxes, n), lbm.LB_COLLOIDS, lbm.PointModel(inv_a=1.4, inv_aL=0.7))
    c.checkpoint_load(buf)
    assert c.steps_taken() == 7


@pytest.mark.parametrize("shape,nboxes,n,kw", [
    ((16, 16, 16), 700, 900, {}),
    ((16, 16, 16), 700, 300, dict(collision="mrt", tau_bulk=0.9)),
    ((13, 30, 13), 600, 500, dict(collision="mrt", tau_bulk=0.9)),
    ((24, 24, 24), 300, 400, {}),
    ((32, 32, 32), 300, 300, dict(collision="mrt", tau_bulk=0.9)),
    ((21, 20, 50), 200, 300, {}),
    ((128, 128, 128), 1, 0, {}),
    ((128, 128, 128), 1, 0, dict(collision="mrt", tau_bulk=0.9)),
    ((128, 128, 128), 1, 300, {}),
    ((160, 100, 190), 1, 400, dict(collision="mrt", tau_bulk=0.9)),
    ((203, 201, 200), 1, 400, dict(collision="mrt", tau_bulk=0.9)),    # cut planes with moving points
])
def test_moment_storage(shape, nboxes, n, kw):
    kind = lbm.LB_COLLOIDS
    a = _run(shape, nboxes, "mom32", n, (64, 4, 1), [11], 70 if n else 0, kind, flow=True, **kw)
    b = _run(shape, nboxes, "mom32", n, None, [11], 70 if n else 0, kind, flow=True, **kw)
    c = _run(shape, nboxes, "mom32", n, None, [3, 4, 1, 3], 70 if n else 0, kind, flow=True, **kw)
    top = max(a[1].abs().max().item(), (a[0] - 1).abs().max().item())
    for x, y in zip(a, b):
        if x.numel():
            assert (x - y).abs().max().item() <= 11 * 32 * EPS * top * (11 if x is a[2] else 1)
    assert all(torch.equal(x, y) for x, y in zip(b, c))


@pytest.mark.parametrize("shape,nboxes,n", [((128, 128, 128), 1, 300), ((160, 100, 190), 1, 200), ((24, 24, 24), 300, 400)])
def test_moment_storage_fixed_points(shape, nboxes, n):
    """The force field laid out once and the velocities handed out, over splits of the run and a change of the sets."""
    a = _run(shape, nboxes, "mom32", n, (64, 4, 1), [11], 70, flow=True)
    b = _run(shape, nboxes, "mom32", n, None, [11], 70, flow=True)
    c = _run(shape, nboxes, "mom32", n, None, [3, 4, 1, 3], 70, flow=True)
    top = max(a[1].abs().max().item(), (a[0] - 1).abs().max().item())
    for x, y in zip(a, b):
        assert (x - y).abs().max().item() <= 11 * 32 * EPS * top * (11 if x is a[2] else 1)
    assert all(torch.equal(x, y) for x, y in zip(b, c))


@pytest.mark.parametrize("storage", ["fp32", "mom32"])
def test_points_in_one_place(storage):
    """More points in a list tile than are staged at once, several tiles of them (all of 900 within 12 x 9 x 7 nodes)."""
    shape, n = (128, 128, 128), 900
    g = np.random.default_rng(11)
    out = []
    for tile in ((64, 4, 1), None):
        g = np.random.default_rng(11)
        pos = torch.tensor(g.uniform(0, 1, (n, 3)) * np.array([12.0, 9.0, 7.0]) + [58.0, 123.0, 60.0], device="cuda")
        frc = torch.tensor(g.normal(scale=1e-6, size=(n, 3)), device="cuda")
        lat = lbm.Lattice(shape, storage, tau=0.7, max_points=n, tile=tile, variant=64 if tile else 0)
        model = lbm.PointModel()
        model.vel_sum = vel = torch.zeros_like(pos)
        lat.add_point_forces(pos, frc, None, lbm.LB_FORCES_STATIC, model)
        lat.step(8)
        _, u = lat.moments()
        lat.sync()
        lat.close()
        out.append((u, vel))
    (ua, va), (ub, vb) = out
    top = ua.abs().max().item()
    if storage == "fp32":
        assert torch.equal(ua, ub)
    assert (ua - ub).abs().max().item() <= 8 * 32 * EPS * top
    assert (va - vb).abs().max().item() <= 8 * 64 * EPS * top * 8
