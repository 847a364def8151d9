"""The MLP loss and gradient at the edges of its sample groups (16 a wave, 128
a pass of a workgroup): against the FP64 oracle."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [15, 16, 33, 127, 128, 129, 1000])
def test_gradient_at_group_edges(B):
    import torch
    from paper_2104_08245_amd import mlp_loss_grad
    rng = np.random.default_rng(B)
    theta = mlp.init_params(rng)
    mean, std = rng.standard_normal(12), 0.5 + rng.random(12)
    x = mean + std * rng.standard_normal((B, 12))
    y = rng.uniform(0.3, 1.0, (B, 2))
    T = lambda a: torch.tensor(np.ascontiguousarray(a, np.float32), device="cuda:0")  # noqa: E731
    grad, loss = torch.full((5122,), 7.0, device="cuda:0"), torch.zeros(1, device="cuda:0")
    mlp_loss_grad(T(theta), T(np.concatenate([mean, std])), T(x), T(y), grad, loss)
    torch.cuda.synchronize()
    f = lambda a: np.asarray(T(a).cpu().numpy(), np.float64)  # noqa: E731
    ref_loss, ref = mlp.loss_and_grad(f(theta), (f(x) - f(mean)) / f(std), f(y))
    # FP32 sums of up to 1,000 samples over three layers
    assert abs(loss.item() - ref_loss) <= 1e-5 * ref_loss
    g = grad.cpu().numpy()
    assert np.linalg.norm(g - ref) <= 1e-5 * np.linalg.norm(ref)
    assert np.abs(g - ref).max() <= 1e-5 * np.abs(ref).max()
