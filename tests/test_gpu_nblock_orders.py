"""More than two blocks whose diagonal blocks' patterns are equal in all, some or
none of the blocks: colours are shared exactly where the patterns are, and cycles
match the oracle."""
import numpy as np
import pytest

from gpu_util import assert_close, log, torch_dev
from paper_2103_07537_amd.inputs import make_system, split_fields

pytestmark = pytest.mark.gpu


def _thin(B, every):
    """B without every `every`-th pair of off-diagonal blocks (i, j), (j, i); their values go to the diagonal."""
    rows = np.repeat(np.arange(B.n_brows), np.diff(B.row_ptr))
    lo, hi = np.minimum(rows, B.col_idx), np.maximum(rows, B.col_idx)
    drop = (rows != B.col_idx) & ((lo.astype(np.int64) * 2654435761 + hi * 40503) // 1000 % every == 0)
    rp = np.zeros(B.n_brows + 1, np.int32)
    rp[1:] = np.cumsum(np.bincount(rows[~drop], minlength=B.n_brows))
    return type(B)(B.n_brows, B.n_bcols, rp, B.col_idx[~drop].copy(), B.vals[~drop].copy())


@pytest.mark.parametrize("thinned", [(), (1,), (1, 3), (2, 3), (1, 2, 3)])
def test_patterns_shared_by_some_blocks(thinned):
    from oracle import amg, nblock
    from paper_2103_07537_amd import mbamg
    t = split_fields(make_system(11, 3, 0.6, seed=5, kappa="lognormal"))
    for f in thinned:
        t.blocks[f][f] = _thin(t.blocks[f][f], 4 if f < 3 else 5)
    ho = nblock.setup(t.blocks, t.dofs, amg.Params(max_coarse=60))
    hg = mbamg.Hierarchy(t.blocks, t.dofs, t.n_vec, max_coarse=60)
    assert hg.num_levels() == len(ho.levels) >= 3
    log(f"  thinned {thinned}: {[int(hg.colours(0, f).max()) + 1 for f in range(4)]} colours")
    pattern = lambda f: (t.blocks[f][f].row_ptr.tobytes(), t.blocks[f][f].col_idx.tobytes())  # noqa: E731
    for f in range(1, 4):
        for e in range(f):
            if pattern(e) == pattern(f):
                assert np.array_equal(hg.colours(0, e), hg.colours(0, f))
    for seed in (1, 2):
        r = np.random.default_rng(seed).standard_normal(t.n_dofs)
        z = torch_dev(np.zeros(t.n_dofs))
        hg.vcycle(torch_dev(r), z)
        assert_close(z.cpu().numpy(), nblock.vcycle(ho, r), 1e-12)
    hg.close()
