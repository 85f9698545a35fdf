"""The FP64 operator read against an FP32 vector (solves whose cycle runs in
FP32), for 1 to 4 dofs per node, sliced and grouped, every block shape: a solve
within one restart cycle converges to the oracle's true residual only if the
operator saw exactly the vector that the solution is combined from."""
import numpy as np
import pytest

from gpu_util import gpu_hierarchy, log, rel, torch_dev
from paper_2103_07537_amd.inputs import leading_components, make_system

pytestmark = pytest.mark.gpu


def _system(d):
    if d == 4:
        return make_system(11, 3, 2.0, seed=5, kappa="lognormal", blk1_scale=0.5, a10_scale=1.5)
    s = make_system(23, 2, 0.7, seed=3, kappa="lognormal", blk1_scale=2.0, a10_scale=0.5)
    return s if d == 3 else leading_components(s, d)


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("form", ["rows", "sliced"])
@pytest.mark.parametrize("shape", ["0", "2"])
def test_fp32_cycle_solves(d, form, shape, monkeypatch):
    from oracle import amg
    monkeypatch.setenv("MBAMG_ROWS_FORM", form)
    monkeypatch.setenv("MBAMG_BLOCK_SHAPE", shape)
    s = _system(d)
    ho = amg.setup(s.blocks, s.dofs, amg.Params(max_coarse=60), n_vec=s.n_vec)
    xo, io = amg.gmres(ho, s.b, rtol=1e-8, restart=30)
    h = gpu_hierarchy(s, max_coarse=60, precision=1)
    x = torch_dev(np.zeros(s.n_dofs))
    info = h.solve(torch_dev(s.b), x, rtol=1e-8)
    h.close()
    got = x.cpu().numpy()
    res = np.linalg.norm(s.b - s.to_scipy() @ got) / np.linalg.norm(s.b)
    log(f"d={d} {form} {shape}: {info['iterations']} iterations, oracle {io.iterations}, residual {res:.2e}")
    # one restart cycle's estimate is the true residual up to FP64 rounding; an operator
    # read off by FP32 rounding would leave about 1e-7
    assert info["converged"] and io.converged
    assert abs(info["iterations"] - io.iterations) <= 1
    assert res <= 1.01e-8
