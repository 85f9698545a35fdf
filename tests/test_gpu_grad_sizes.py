"""The network's loss and gradient at batch sizes on the edges of its tiles
(64 rows per workgroup step, at most 256 workgroups) against the
bfloat16-emulating oracle.  The last row's target is far off, so its share
dominates the sums and a dropped row or partial cannot hide."""
import numpy as np
import pytest

from gpu_util import rel, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 63, 64, 65, 577, 64 * 256, 64 * 256 + 1])
def test_gradient_at_tile_edges(n):
    import torch
    from oracle import learned
    from paper_2103_07537_amd import mbamg
    rng = np.random.default_rng(n)
    th = learned.init_params(3)
    th[4992:5122] = rng.standard_normal(130) * 0.3
    th = th.astype(np.float32)
    X = rng.standard_normal((n, 12)).astype(np.float32)
    T = rng.uniform(0.3, 0.8, (n, 2)).astype(np.float32)
    T[-1] = np.sqrt(n) * 10.0
    grad = torch.full((5122,), float("nan"), dtype=torch.float32, device="cuda")
    loss = torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
    mbamg.mlp_loss_grad(torch_dev(th), torch_dev(X), torch_dev(T), grad, loss)
    L, g = learned.loss_grad(th.astype(np.float64), X.astype(np.float64), T.astype(np.float64), emulate=True)
    assert abs(loss.item() - L) <= 1e-5 * abs(L)
    # one bfloat16 rounding that falls the other way in FP32 than in FP64 is 2^-8 of that value
    assert rel(grad.cpu().numpy(), g) <= 2.0 ** -8
