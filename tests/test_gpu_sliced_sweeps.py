"""Sliced levels colour by colour, whose last launch leaves out the undamped
iterate where no later launch reads it: one to three inner sweeps, one and two
outer ones, against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_close, gpu_hierarchy, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


# tolerance: the oracle's sums in another order (as in the other V-cycle parity tests)
@pytest.mark.parametrize("dim,n", [(2, 37), (3, 11)])
@pytest.mark.parametrize("bgs", [1, 2])
@pytest.mark.parametrize("inner", [1, 2, 3])
@pytest.mark.parametrize("split", ["1", "2"])
def test_sliced_sweeps_match_the_oracle(dim, n, bgs, inner, split, monkeypatch):
    from oracle import amg
    monkeypatch.setenv("MBAMG_ROWS_FORM", "sliced")
    monkeypatch.setenv("MBAMG_SLICE_SPLIT", split)
    s = make_system(n, dim, 0.7, seed=3, kappa="lognormal", blk1_scale=1.7, a10_scale=0.6)
    kw = dict(max_coarse=60, bgs_sweeps=bgs, inner_sweeps=inner, omega=0.7)
    ho = amg.setup(s.blocks, s.dofs, amg.Params(**kw), n_vec=s.n_vec)
    h = gpu_hierarchy(s, **kw)
    r = np.random.default_rng(n).standard_normal(s.n_dofs)
    z = torch_dev(np.zeros(s.n_dofs))
    for _ in range(2):   # the second cycle finds the first one's buffers
        h.vcycle(torch_dev(r), z)
        assert_close(z.cpu().numpy(), amg.vcycle(ho, r), 1e-12)
    h.close()
