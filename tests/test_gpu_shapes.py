"""Block shapes: levels whose blocks are a multiple of the identity on the
vector components (and equal in last column and last row) store only the entries
that determine a block.  The sums run over the same nonzero terms in the same
order, so cycles, applies and solves are bit for bit those of the full storage;
and systems whose blocks miss one or both conditions, in one block of the finest
level alone or everywhere, match the oracle."""
import numpy as np
import pytest

from gpu_util import assert_close, gpu_hierarchy, log, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


def weights_fn(level, n_agg, F):
    k = np.arange(n_agg)
    return 0.1 + 0.6 * ((k * 37 + level) % 11) / 10.0, 0.5 + 0.5 * ((k * 13 + 3 * level) % 7) / 6.0


CASES = {
    "3d-11": lambda: make_system(11, 3, 2.0, seed=5, kappa="lognormal", blk1_scale=1.7, a10_scale=0.6),
    "2d-37": lambda: make_system(37, 2, 0.7, seed=3, kappa="lognormal"),
}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("form", ["fp64", "fp32", "weighted"])
@pytest.mark.parametrize("layout", ["grouped", "sliced-1", "sliced-2"])
def test_shaped_storage_is_bit_identical_to_full(case, form, layout, monkeypatch):
    s = CASES[case]()
    kw = dict(max_coarse=60, precision=1 if form == "fp32" else 0)
    if form == "weighted":
        kw.update(weights=weights_fn, judge=0)
    if layout != "grouped":
        monkeypatch.setenv("MBAMG_ROWS_FORM", "sliced")
        monkeypatch.setenv("MBAMG_SLICE_SPLIT", layout[-1])
    r = torch_dev(np.random.default_rng(1).standard_normal(s.n_dofs))
    got = {}
    for shape in ("0", "1", "2"):
        monkeypatch.setenv("MBAMG_BLOCK_SHAPE", shape)
        h = gpu_hierarchy(s, **kw)
        z, w, x = (torch_dev(np.zeros(s.n_dofs)) for _ in range(3))
        h.vcycle(r, z)
        h.apply(r, w)
        info = h.solve(torch_dev(s.b), x, rtol=1e-8)
        got[shape] = (z.cpu().numpy(), w.cpu().numpy(), x.cpu().numpy(), info["iterations"])
        h.close()
    for shape in ("1", "2"):
        for a, b in zip(got[shape][:3], got["0"][:3]):
            assert np.array_equal(a, b)
        assert got[shape][3] == got["0"][3]


def _break(s, what):
    """One condition broken: `scaled` in the last column, `full` in the leading part; in every block of A00,
    in the last block of A11 alone, or in the coupling A01."""
    rng = np.random.default_rng(9)
    kind, where = what.split("-")
    B = {"all": s.blocks[0][0], "last": s.blocks[1][1], "coupling": s.blocks[0][1]}[where]
    B.vals = B.vals.copy()
    sel = slice(None) if where != "last" else slice(-1, None)
    d = B.vals.shape[1]
    scale = 0.01 * np.abs(B.vals).max()
    if kind == "scaled":
        B.vals[sel, :d - 1, d - 1] += scale * rng.uniform(0.5, 1.0, B.vals[sel, :d - 1, d - 1].shape)
    else:
        B.vals[sel, 0, 0] *= 1.01
        B.vals[sel, 0, 1] += scale * rng.uniform(0.5, 1.0, B.vals[sel, 0, 1].shape)
    return s


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("layout", ["grouped", "sliced-1", "sliced-2"])
@pytest.mark.parametrize("what", ["scaled-all", "scaled-last", "scaled-coupling", "full-all", "full-last",
                                  "full-coupling"])
def test_systems_that_miss_a_condition_match_the_oracle(dim, layout, what, monkeypatch):
    from oracle import amg
    s = _break(make_system(10, 3, 1.0, seed=5, kappa="lognormal") if dim == 3 else
               make_system(33, 2, 0.7, seed=3, kappa="lognormal"), what)
    if layout != "grouped":
        monkeypatch.setenv("MBAMG_ROWS_FORM", "sliced")
        monkeypatch.setenv("MBAMG_SLICE_SPLIT", layout[-1])
    ho = amg.setup(s.blocks, s.dofs, amg.Params(max_coarse=60), n_vec=s.n_vec)
    r = np.random.default_rng(2).standard_normal(s.n_dofs)
    ref = amg.vcycle(ho, r)
    for precision, tol in ((0, 1e-12), (1, 1e-5)):
        hg = gpu_hierarchy(s, max_coarse=60, precision=precision)
        assert hg.num_levels() == len(ho.levels) >= 3
        log(f"dim={dim} layout={layout} what={what} precision={precision}")
        z = torch_dev(np.zeros(s.n_dofs))
        hg.vcycle(torch_dev(r), z)
        assert_close(z.cpu().numpy(), ref, tol)
        w = torch_dev(np.zeros(s.n_dofs))
        hg.apply(torch_dev(r), w)
        a = amg.apply_A(ho.levels[0], r)
        assert np.max(np.abs(w.cpu().numpy() - a)) <= 1e-13 * np.max(np.abs(a))
        hg.close()
