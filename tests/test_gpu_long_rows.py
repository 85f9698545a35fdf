"""Rows far longer than the rest in the grouped form: hubs coupled to 100, 700 and
1500 of 2025 nodes, so that a row's blocks are put in order by a few lanes, by a
whole wavefront, or (more than 1024) in one linear pass."""
import numpy as np
import pytest

from gpu_util import assert_close, gpu_hierarchy, log, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


def _with_hubs(s, hubs):
    """hubs: {node: number of other nodes it is coupled to}, in both diagonal blocks, weakly and both ways."""
    import scipy.sparse as sp
    rng = np.random.default_rng(11)
    d = s.dofs[0]
    rows, cols = [], []
    for hub, k in hubs.items():
        others = rng.choice(np.setdiff1d(np.arange(s.N), list(hubs)), size=k, replace=False)
        rows += [np.full(k, hub), others]
        cols += [others, np.full(k, hub)]
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    for f in range(2):
        B = s.blocks[f][f]
        scale = 1e-5 * np.abs(B.vals).max()
        have = np.repeat(np.arange(s.N), np.diff(B.row_ptr))
        key = np.concatenate([have.astype(np.int64) * s.N + B.col_idx, rows.astype(np.int64) * s.N + cols])
        v = np.concatenate([B.vals, scale * rng.uniform(0.5, 1.0, (len(rows), 1, 1)) * np.eye(d)])
        u, where = np.unique(key, return_inverse=True)
        vals = np.zeros((len(u), d, d))
        np.add.at(vals, where, v)
        rp = np.zeros(s.N + 1, np.int32)
        rp[1:] = np.cumsum(np.bincount(u // s.N, minlength=s.N))
        s.blocks[f][f] = type(B)(s.N, s.N, rp, (u % s.N).astype(np.int32), vals)
    return s


@pytest.mark.parametrize("group", ["4", "16", "64", None])
@pytest.mark.parametrize("precision", [0, 1])
def test_long_rows_match_the_oracle(group, precision, monkeypatch):
    from oracle import amg
    s = _with_hubs(make_system(45, 2, 0.7, seed=3, kappa="lognormal"), {7: 100, 1000: 700, 2000: 1500})
    kw = dict(max_coarse=60, theta=0.05)
    ho = amg.setup(s.blocks, s.dofs, amg.Params(**kw), n_vec=s.n_vec)
    if group:
        monkeypatch.setenv("MBAMG_SWEEP_GROUP", group)
    hg = gpu_hierarchy(s, precision=precision, **kw)
    assert hg.num_levels() == len(ho.levels) >= 3
    assert np.diff(hg.level_block(0, 0, 0)[0]).max() > 1500 and np.diff(hg.level_block(1, 0, 0)[0]).max() > 64
    z = torch_dev(np.zeros(s.n_dofs))
    for seed in (1, 2):
        r = np.random.default_rng(seed).standard_normal(s.n_dofs)
        hg.vcycle(torch_dev(r), z)
        assert_close(z.cpu().numpy(), amg.vcycle(ho, r), 1e-12 if precision == 0 else 1e-5)
    w = torch_dev(np.zeros(s.n_dofs))
    hg.apply(torch_dev(r), w)
    a = amg.apply_A(ho.levels[0], r)
    assert np.max(np.abs(w.cpu().numpy() - a)) <= 1e-13 * np.max(np.abs(a))
    hg.close()
