"""Column indices as 16-bit offsets per slot against 32-bit ones: the same bits in
every result, for 1 to 4 dofs per node, FP64 and FP32; forms that keep 32 bits
(split slices, the full-node smoother, transfers); and a node order that spreads a
slot's columns over more than 16 bits, which keeps 32 too."""
import numpy as np
import pytest

from gpu_util import gpu_hierarchy, torch_dev
from paper_2103_07537_amd.inputs import leading_components, make_system

pytestmark = pytest.mark.gpu


def _system(d):
    if d == 4:
        return make_system(11, 3, 2.0, seed=5, kappa="lognormal", blk1_scale=0.5, a10_scale=1.5)
    s = make_system(23, 2, 0.7, seed=3, kappa="lognormal", blk1_scale=2.0, a10_scale=0.5)
    return s if d == 3 else leading_components(s, d)


def _results(s, monkeypatch, short, **kw):
    monkeypatch.setenv("MBAMG_ROWS_FORM", "sliced")
    monkeypatch.setenv("MBAMG_COL16", short)
    h = gpu_hierarchy(s, max_coarse=60, **kw)
    rng = np.random.default_rng(7)
    r, z, w = (torch_dev(v) for v in (rng.standard_normal(s.n_dofs), np.zeros(s.n_dofs), np.zeros(s.n_dofs)))
    h.vcycle(r, z)
    h.apply(r, w)
    h.close()
    return z.cpu().numpy(), w.cpu().numpy()


FORMS = {
    "plain": {},
    "fp32": dict(precision=1),
    "full-node": dict(smoother=1),
    "smoothed": dict(omega_p=0.5),
}


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("split", ["1", "2", "16"])
def test_short_columns_change_nothing(d, form, split, monkeypatch):
    monkeypatch.setenv("MBAMG_SLICE_SPLIT", split)
    s = _system(d)
    a = _results(s, monkeypatch, "0", **FORMS[form])
    b = _results(s, monkeypatch, "1", **FORMS[form])
    for x, y in zip(a, b):
        assert np.all(np.isfinite(x)) and x.tobytes() == y.tobytes()


def test_spread_columns_keep_32_bits(monkeypatch):
    s = leading_components(make_system(400, 2, 0.7, seed=3), 1)
    p = np.random.default_rng(3).permutation(s.N)
    for row in s.blocks:
        for k, a in enumerate(row):
            m = a.to_scipy()[p][:, p].tocsr()
            m.sort_indices()
            row[k] = type(a)(s.N, s.N, m.indptr.astype(np.int32), m.indices.astype(np.int32),
                             m.data.reshape(-1, 1, 1))
    a = _results(s, monkeypatch, "0")
    b = _results(s, monkeypatch, "1")
    for x, y in zip(a, b):
        assert np.all(np.isfinite(x)) and x.tobytes() == y.tobytes()
