"""Point lists of few points in many tiles (the blocks of the build then follow from the tiles, not the points): every
node that a stencil reaches finds its points, so the force density sums to the forces and their first moments to the
torques: 64 FP32 products a point, each to 2 ** -24."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


@pytest.mark.parametrize("shape,storage,tile,variant", [
    ((16, 256, 256), "mom32", (64, 2, 2), 64),         # 4096 tiles: the fewest blocks
    ((128, 256, 256), "mom32", (64, 2, 2), 64),        # 32768, the last before more
    ((256, 256, 256), "mom32", (64, 2, 2), 64),        # 65536
    ((131, 255, 300), "mom32", (16, 4, 4), 0),         # 65472, ragged
    ((320, 384, 384), "fp16", (64, 2, 2), 64),         # 184320
])
def test_few_points_in_many_tiles(shape, storage, tile, variant):
    ext = np.array(shape[::-1], dtype=np.float64)
    pos = np.array([[1.3, 2.2, 3.9], [130.5, 77.1, 9.4], [200.2, 200.7, 1.9]])
    pos = np.concatenate([pos, [ext - 3.6]])         # the last tiles too
    frc = np.random.default_rng(2).normal(scale=1e-6, size=pos.shape)
    lat = lbm.Lattice(shape, storage, tau=0.7, max_points=len(pos), tile=tile, variant=variant,
                      fp16_exponent=20 if storage == "fp16" else 0)
    for _ in range(2):                                 # a second build on the first one's counters
        lat.clear_forces()
        lat.add_point_forces(torch.tensor(pos, device="cuda"), torch.tensor(frc, device="cuda"))
        r, d = lat.diagnostics()
        assert r == lbm.LB_OK
        assert np.abs(d[0, 4:7] - frc.sum(0)).max() <= 64 * 2.0 ** -24 * np.abs(frc).sum()
        assert np.abs(d[0, 7:10] - np.cross(pos, frc).sum(0)).max() <= 64 * 2.0 ** -24 * np.abs(frc).sum() * 2 * ext.max()
