"""Steps of one call hand their points' records on to each other; steps of separate calls do not.  Both
must give the same bits: several colloid sets (with a fixed set and the network among them), noise,
FP16 exponents that change from step to step, batches of boxes, points that leave their windows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm, mobility  # noqa: E402


def _run(calls, storage, nboxes, kT, speed):
    shape = (12, 10, 20)
    g = np.random.default_rng(11)
    ext = np.array(shape[::-1], dtype=np.float64)
    lat = lbm.Lattice(shape, storage, nboxes=nboxes, tau=0.8, zero_net_force=True, max_points=60, kT=kT, seed=9,
                      fp16_exponent=14)   # FP16: forces of 3e-3 overflow at the rest state's 2^30
    out = []
    for k, (n, kind) in enumerate(((21, lbm.LB_COLLOIDS), (9, lbm.LB_FORCES_STATIC), (30, lbm.LB_COLLOIDS))):
        pos = torch.tensor(g.uniform(0, 1, (n, 3)) * ext, device="cuda")
        frc = torch.tensor(g.normal(scale=speed, size=(n, 3)), device="cuda")
        box = torch.tensor(g.integers(0, nboxes, n).astype(np.int32), device="cuda")
        vel = torch.zeros_like(pos)
        if k == 2:
            model = mobility.load(mobility.DEFAULT_NET).model(8.5, vel_sum=vel)
        else:
            model = lbm.PointModel(inv_a=8.5, inv_aL=0.77, vel_out=vel)
        lat.add_point_forces(pos, frc, box, kind, model)
        out += [pos, vel]
    for n in calls:
        lat.step(n)
    rho, u = lat.moments()
    lat.sync()
    return out + [rho, u]


@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16", "mom32"])
@pytest.mark.parametrize("nboxes,kT", [(1, 0.0), (3, 0.0), (1, 1e-6)])
def test_one_call_equals_many(storage, nboxes, kT):
    if storage == "mom32" and kT > 0:
        pytest.skip("moment storage takes no noise")
    # forces that move a colloid by up to a node in a few steps
    one = _run([22], storage, nboxes, kT, 3e-3)
    for calls in ([1] * 22, [3, 3, 16], [5, 1, 2, 14]):
        for a, b in zip(one, _run(calls, storage, nboxes, kT, 3e-3)):
            assert torch.equal(a, b)
