"""The network kernels at the edges of their split into batches of 16 samples and blocks: one sample,
a partial and a whole batch, the last count one block serves and the first for two, several
batches per block, and more batches than blocks.  Against the FP64 oracle; FP32 dot products of at
most 64 terms and sample sums give a few 1e-6 of the largest gradient, bounded at 1e-4 (gradient,
with cancellation between samples) and 2e-6 (outputs of order one)."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_0707_1299_amd import lbm  # noqa: E402


@pytest.mark.parametrize("n", [1, 15, 16, 17, 35, 36, 531, 4111, 16401])
def test_forward_and_gradient(n):
    g = np.random.default_rng(n)
    master = (omlp.init_params(1) + g.normal(scale=0.05, size=omlp.NPARAM)).astype(np.float32)
    X = g.uniform(-1, 1, size=(n, 4)).astype(np.float32)
    y = (0.3 * np.sin(2 * X[:, 0]) * np.cos(X[:, 1]) + 0.1 * X[:, 3] + 0.2).astype(np.float32)
    w16 = torch.zeros(lbm.LBML_NPARAM, dtype=torch.int16, device="cuda")
    lbm.lbml_round_bf16(torch.tensor(master, device="cuda"), w16)
    xd, yd = torch.tensor(X, device="cuda"), torch.tensor(y, device="cuda")
    # guard words behind every output and behind the work memory stay as they are
    out, grad = torch.full((n + 8,), 7.0, device="cuda"), torch.full((lbm.LBML_NPARAM + 8,), 7.0, device="cuda")
    loss, work = torch.full((9,), 7.0, device="cuda"), torch.full((lbm.lbml_work_floats(n) + 8,), 7.0, device="cuda")
    lbm.lbml_forward(w16, xd, out)
    lbm.lbml_loss_grad(w16, xd, yd, grad, loss, work)
    for t, used in ((out, n), (grad, lbm.LBML_NPARAM), (loss, 1), (work, lbm.lbml_work_floats(n))):
        assert bool((t[used:] == 7.0).all())
    ref, _ = omlp.forward(master, X)
    assert np.abs(out[:n].cpu().numpy() - ref).max() <= 2e-6 * max(1.0, np.abs(ref).max())
    l_ref, g_ref = omlp.loss_and_grad(master, X, y, round_bf16=True)
    assert abs(loss[0].item() - l_ref) <= 1e-5 * l_ref
    got = grad[:lbm.LBML_NPARAM].cpu().numpy().astype(np.float64)
    assert np.abs(got - g_ref).max() <= 1e-4 * np.abs(g_ref).max()
