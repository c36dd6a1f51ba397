"""Cost-model kernels at the sample counts where their tiling can go wrong
(waves of 16 samples, workgroups of 64, one to several tiles per wave),
against the FP64 NumPy oracle. Tolerance: FP32 products and sums over at most
64 + 12 + 64 terms per layer, about 1e-6 of the largest value; the gradient's
partial sums run over up to 16 * tiles samples, 1e-5."""
import numpy as np
import pytest

from oracle import mlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1000, 32768, 32769])
def test_predict_gradient_and_norm_at_tile_edges(n):
    rng = np.random.default_rng(n)
    X = (rng.standard_normal((n, 12)) * rng.uniform(0.5, 3.0, 12) + rng.uniform(-2, 2, 12)).astype(np.float32)
    t = (np.sin(X[:, 0]) + 0.3 * X[:, 1] * X[:, 2] + 2.0).astype(np.float32)
    cm = fea.CostModel(seed=21)
    Xd, td = torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda()
    cm.fit_norm(Xd)
    mean = X.astype(np.float64).mean(axis=0).astype(np.float32).astype(np.float64)
    sd = X.astype(np.float64).std(axis=0)
    scale = np.where(sd > 1e-12, sd, 1.0).astype(np.float32).astype(np.float64)
    theta = cm.params().astype(np.float64)
    y_ref, _ = mlp.forward(theta, X.astype(np.float64), mean, scale)
    y = cm.predict(Xd).cpu().numpy()
    assert np.abs(y - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max())
    g, loss = cm.grad(Xd, td)
    l_ref, g_ref = mlp.loss_grad(theta, X.astype(np.float64), t.astype(np.float64), mean, scale)
    assert abs(float(loss.item()) - l_ref) <= 1e-5 * l_ref
    assert np.abs(g.cpu().numpy() - g_ref).max() <= 1e-5 * np.abs(g_ref).max()
    g2, _ = cm.grad(Xd, td)
    assert torch.equal(g, g2)
