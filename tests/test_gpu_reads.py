"""Moments and diagnostics between steps on the tile and block order that reads take, against a context that names the plain
tile (whose reads keep it): the fields bit for bit, the sums of the diagnostics to their FP64 rounding (moment storage with
marching steps: to the rounding of its gathered sums).  One shape per rule: rows on and off the cache lines, 128-node tiles
that rows do not fill, marching lattices with and without points."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


def _reads(shape, storage, nboxes, npts, tile):
    g = np.random.default_rng(5)
    lat = lbm.Lattice(shape, storage, nboxes=nboxes, tau=0.7, max_points=npts, tile=tile,
                      fp16_exponent=16 if storage == "fp16" else 0)
    lat.set_equilibrium(torch.tensor(1 + g.uniform(-1e-3, 1e-3, (nboxes,) + shape), device="cuda"),
                        torch.tensor(g.uniform(-1e-3, 1e-3, (nboxes, 3) + shape), device="cuda"))
    if npts:
        pos = torch.tensor(g.uniform(0, 1, (npts, 3)) * np.array(shape[::-1], dtype=np.float64), device="cuda")
        lat.add_point_forces(pos, torch.tensor(g.normal(scale=1e-6, size=(npts, 3)), device="cuda"),
                             torch.tensor(g.integers(0, nboxes, npts).astype(np.int32), device="cuda"))
    lat.step(2)
    rho, u = lat.moments()
    r, d = lat.diagnostics()
    assert r == lbm.LB_OK
    lat.step(1)
    rho1, u1 = lat.moments(rho=False)
    lat.sync()
    return rho, u, u1, d


@pytest.mark.parametrize("shape,storage,nboxes,npts", [
    ((9, 10, 160), "fp16", 1, 0), ((9, 10, 160), "fp16", 1, 20), ((5, 6, 300), "fp16", 2, 0), ((9, 10, 256), "fp16", 1, 0),
    ((24, 24, 24), "fp32", 300, 0), ((24, 24, 24), "fp32", 300, 200), ((96, 96, 96), "fp32", 1, 0),
    ((20, 64, 300), "fp32", 1, 7), ((200, 200, 192), "fp32", 1, 0), ((200, 200, 192), "fp32", 1, 9),
    ((12, 10, 101), "fp64", 2, 5), ((9, 8, 64), "fp64", 1, 0), ((16, 12, 300), "mom32", 1, 5), ((128, 128, 128), "mom32", 1, 0),
])
def test_reads_as_on_the_plain_tile(shape, storage, nboxes, npts):
    plain = (128, 1, 2) if storage == "mom32" and shape[2] >= 128 else (64, 2, 2) if shape[2] >= 64 else (16, 4, 4)
    a, b = _reads(shape, storage, nboxes, npts, None), _reads(shape, storage, nboxes, npts, plain)
    marched = storage == "mom32"
    for x, y in zip(a[:3], b[:3]):
        if x is not None:
            assert (x - y).abs().max().item() <= (3 * 32 * 2.0 ** -24 * 2e-3 if marched else 0.0)
    N = shape[0] * shape[1] * shape[2]
    size = np.array([4e-3] * 4 + [1e-5] * 3 + [1e-5 * max(shape)] * 3 + [4e-3, 0, 0]) * N      # a bound on each sum's terms
    size[10] = 4e-3
    eps = 3 * 32 * 2.0 ** -24 if marched else 64 * 2.0 ** -53
    assert (np.abs(a[3] - b[3]) <= eps * size + 0).all()
