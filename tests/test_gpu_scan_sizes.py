"""The prefix sums of the setup where their number of 1024-item blocks changes:
every array they size or place (aggregates, members, patterns of the coarse
operators) against the CPU oracle, as integers."""
import numpy as np
import pytest

from gpu_util import gpu_hierarchy, oracle_params
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


# nodes: 4, 961, 1024 (one block), 1089 (two), 2025, 4096 (four blocks exactly), 4225
@pytest.mark.parametrize("n", [2, 31, 32, 33, 45, 64, 65])
def test_setup_arrays_at_scan_block_edges(n):
    from oracle import amg
    s = make_system(n, 2, 0.5, seed=n)
    ho = amg.setup(s.blocks, s.dofs, oracle_params(max_coarse=40))
    hg = gpu_hierarchy(s, max_coarse=40)
    assert hg.num_levels() == len(ho.levels)
    for l, lev in enumerate(ho.levels):
        assert hg.level_nodes(l) == lev.n
        if l + 1 < len(ho.levels):
            assert np.array_equal(hg.aggregates(l), lev.agg)
        if l > 0:
            for f in range(2):
                for g in range(2):
                    rp, ci, _ = hg.level_block(l, f, g)
                    assert np.array_equal(rp, lev.A[f][g].rp) and np.array_equal(ci, lev.A[f][g].ci)
