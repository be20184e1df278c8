"""The library's own choice of tile and variant against the plain tile (64 x 2 x 2, 32 x 4 x 2 or 16 x 4 x 4 with variant
0), one shape per rule of the choice: the fields of a run with fixed forces are the same bit for bit
(each node's arithmetic does not depend on its tile), the interpolated velocity to the rounding
of its partial sums.  Checkpoints of the plain tile still load, those of any other tile are refused."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


def _run(shape, storage, tile, kw, npts, steps=6, nboxes=1):
    g = np.random.default_rng(5)
    ext = np.array(shape[::-1], dtype=np.float64)
    pos = torch.tensor(g.uniform(0, 1, (npts, 3)) * ext, device="cuda")
    frc = torch.tensor(g.normal(scale=1e-6, size=(npts, 3)), device="cuda")
    box = torch.tensor(g.integers(0, nboxes, npts).astype(np.int32), device="cuda")
    lat = lbm.Lattice(shape, storage, nboxes=nboxes, tau=0.7, max_points=npts, tile=tile, **kw)
    vel = torch.zeros_like(pos)
    lat.add_point_forces(pos, frc, box, lbm.LB_FORCES_STATIC, lbm.PointModel(vel_out=vel))
    lat.step(steps)
    rho, u = lat.moments()
    lat.sync()
    return rho, u, vel


@pytest.mark.parametrize("shape,storage,kw,npts,nboxes", [
    ((33, 40, 101), "fp32", {}, 20, 1),                        # rows of 65 .. 128 nodes
    ((60, 50, 101), "fp32", dict(collision="bgk"), 20, 1),     # ... rows off the cache lines, general operator
    ((40, 64, 320), "fp32", {}, 9, 1),                         # rows of 192 and more, last tile mostly empty
    ((34, 64, 256), "fp32", {}, 9, 1),                         # one row per block
    ((34, 64, 256), "fp32", {}, 3000, 1),                      # the same with many points
    ((12, 48, 256), "fp64", {}, 9, 1),
    ((12, 10, 48), "fp32", {}, 300, 30),                       # rows of 33 .. 63 nodes
    ((48, 64, 128), "mom32", {}, 9, 1),
    ((48, 64, 128), "fp16", {}, 9, 1),                         # two nodes per lane, whole waves
    ((16, 16, 16), "fp16", {}, 200, 200),                      # a batch of FP16 boxes
    ((64, 64, 96), "fp32", dict(kT=1e-5, seed=4), 9, 1),       # thermal
    ((9, 9, 9), "fp32", {}, 5, 1),
    ((14, 18, 25), "fp64", {}, 9, 1),                          # rows of 17 .. 31 nodes
    ((14, 18, 29), "mom32", {}, 9, 1),
    ((14, 18, 26), "fp16", {}, 9, 1),
    ((20, 16, 31), "fp16", {}, 9, 1),                          # one node per lane, small
    ((20, 21, 75), "fp64", dict(kT=1e-5, seed=4), 9, 1),       # thermal, 32-node tiles
    ((20, 21, 36), "fp64", dict(kT=1e-5, seed=4), 9, 1),       # ... the last too empty
])
def test_same_fields_as_plain_tile(shape, storage, kw, npts, nboxes):
    plain = (64, 2, 2) if shape[2] >= 64 else (32, 4, 2) if shape[2] >= 32 else (16, 4, 4)
    a = _run(shape, storage, None, kw, npts, nboxes=nboxes)
    b = _run(shape, storage, plain, kw, npts, nboxes=nboxes)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    top = b[1].abs().max().item()
    assert (a[2] - b[2]).abs().max().item() <= (1e-14 if storage == "fp64" else 1e-6) * top


def test_checkpoint_of_the_plain_tile_loads():
    shape = (20, 12, 101)
    g = np.random.default_rng(8)
    ext = np.array(shape[::-1], dtype=np.float64)
    p0, f0 = g.uniform(0, 1, (11, 3)) * ext, g.normal(scale=1e-5, size=(11, 3))

    def make(tile, pos):
        lat = lbm.Lattice(shape, "fp64", tau=0.7, max_points=11, tile=tile)
        p = torch.tensor(pos, device="cuda")
        lat.add_point_forces(p, torch.tensor(f0, device="cuda"), None, lbm.LB_COLLOIDS,
                             lbm.PointModel(inv_a=2.0, inv_aL=0.7))
        return lat, p

    old, p = make((64, 2, 2), p0)
    old.step(7)
    buf = torch.empty(old.checkpoint_bytes() + 256, dtype=torch.uint8, device="cuda")
    old.checkpoint_save(buf)
    saved = p.cpu().numpy()
    old.step(9)
    new, q = make(None, saved)
    new.checkpoint_load(buf)
    new.step(9)
    _, ua = old.moments()
    _, ub = new.moments()
    old.sync()
    assert new.steps_taken() == 16
    assert (ua - ub).abs().max().item() <= 1e-13 * ua.abs().max().item()
    assert (p - q).abs().max().item() <= 1e-12
    other, _ = make((32, 4, 2), saved)
    with pytest.raises(lbm.LBError):
        other.checkpoint_load(buf)
