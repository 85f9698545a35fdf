"""A caller that wants no limit on the number of levels passes the largest one:
the setup takes no memory for levels that do not exist, and builds the same
hierarchy as with the default limit."""
import numpy as np
import pytest

from gpu_util import gpu_hierarchy, log, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
def test_no_limit_on_the_levels_costs_nothing(dim):
    import torch
    s = make_system(37, 2, 0.7, seed=3) if dim == 2 else make_system(11, 3, 2.0, seed=5, kappa="lognormal")
    r = torch_dev(np.random.default_rng(1).standard_normal(s.n_dofs))
    got = []
    for levels in (10, 2 ** 31 - 1):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        h = gpu_hierarchy(s, max_coarse=60, max_levels=levels)
        taken = free - torch.cuda.mem_get_info()[0]
        log(f"  dim={dim} max_levels={levels}: {h.num_levels()} levels, {taken / 2 ** 20:.0f} MiB taken")
        assert h.num_levels() >= 3 and taken < 2 ** 30
        z = torch_dev(np.zeros(s.n_dofs))
        h.vcycle(r, z)
        got.append(z.cpu().numpy().tobytes())
        h.close()
    assert got[0] == got[1]
