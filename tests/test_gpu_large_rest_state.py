"""The rest state of a lattice whose population copies hold 2 ** 32 words and more (34 GB of workspace) on memory that held
something else: every node is at rest and finite."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


def test_rest_state_of_a_large_lattice():
    shape = (640, 640, 560)            # 19 FP32 planes: 4.36e9 words a copy
    n = lbm.lb_workspace_bytes(lbm.make_params(shape, "fp32", tau=0.7))
    if torch.cuda.mem_get_info()[0] < n + (4 << 30):
        pytest.skip("needs %.0f GB of device memory" % (n / 1e9 + 4))
    dirty = torch.full((n + 256,), 255, dtype=torch.uint8, device="cuda")     # NaN in every word
    where = dirty.data_ptr()
    del dirty
    lat = lbm.Lattice(shape, "fp32", tau=0.7)
    assert lat.workspace.data_ptr() == where       # the allocator gave the same memory back
    r, d = lat.diagnostics()
    lat.step(1)
    r2, d2 = lat.diagnostics()
    lat.close()
    del lat
    torch.cuda.empty_cache()
    for status, v in ((r, d), (r2, d2)):
        assert status == lbm.LB_OK and v[0, 11] == 0 and v[0, 12] == 0
        assert (v[0, :11] == 0).all()
