"""The gradient's two ways of leaving partial sums (one per wavefront on grids of up
to 64 workgroups of 64 rows, one per workgroup above) on both sides of the line:
against the bfloat16-emulating oracle, and both entry points bit for bit."""
import numpy as np
import pytest

from gpu_util import rel, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 129, 64 * 64 - 1, 64 * 64, 64 * 64 + 1, 64 * 65])
def test_gradient_on_both_sides_of_the_line(n):
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
    args = [torch_dev(v) for v in (th, X, T)]
    out = [[torch.full((k,), float("nan"), dtype=torch.float32, device="cuda") for k in (5122, 1)] for _ in range(2)]
    mbamg.mlp_loss_grad(*args, *out[0])
    mbamg.mlp_loss_grad_noalloc(*args, *out[1])
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    L, g = learned.loss_grad(th.astype(np.float64), X.astype(np.float64), T.astype(np.float64), emulate=True)
    assert abs(out[0][1].item() - L) <= 1e-5 * abs(L)
    # one bfloat16 rounding that falls the other way in FP32 than in FP64 is 2^-8 of that value
    assert rel(out[0][0].cpu().numpy(), g) <= 2.0 ** -8
