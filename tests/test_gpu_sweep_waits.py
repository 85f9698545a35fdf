"""The sweeps' waits under full load: a 2D system whose second level has more
workgroups of 3 x 3 FP64 rows than the chip holds at once, all polling, over
hundreds of solver iterations.  Every restart has to reduce the residual, and
repeated restarts from the same iterate give the same one bit for bit (a wait
that runs out leaves NaN behind)."""
import numpy as np
import pytest

from gpu_util import gpu_hierarchy, log, torch_dev
from paper_2103_07537_amd.inputs import leading_components, make_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [3, 1])
@pytest.mark.parametrize("precision", [0, 1])
def test_waits_of_many_workgroups_end(d, precision):
    import torch
    s = make_system(900, 2, 0.5, seed=2, kappa="lognormal")
    if d != 3:
        s = leading_components(s, d)
    h = gpu_hierarchy(s, max_iters=30, precision=precision)
    assert h.num_levels() >= 3 and h.level_nodes(1) > 65536
    b = torch_dev(s.b)
    x, first = torch.zeros_like(b), None
    last = np.inf
    for k in range(24):
        if k % 4 == 0:
            x.zero_()
            last = 1.0
        info = h.solve(b, x, rtol=1e-14)
        assert torch.isfinite(x).all() and info["rel_residual"] < last
        last = info["rel_residual"]
        if k % 4 == 0:
            first = x.clone() if first is None else first
            assert torch.equal(x, first)
    log(f"  d={d} precision={precision}: rel {last:.2e} after 4 restarts")
    h.close()
