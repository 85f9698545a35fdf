"""Which layout a level takes, from what the setup reports with MBAMG_VERBOSE: the
comparisons of layouts with each other (16-bit columns against 32, shaped blocks
against full ones, grouped levels against sliced) would pass if one were never
chosen."""
import re

import numpy as np
import pytest

from gpu_util import gpu_hierarchy, log
from paper_2103_07537_amd.inputs import leading_components, make_system

pytestmark = pytest.mark.gpu


def _layout(s, capfd, monkeypatch, **kw):
    """Per level: ("sliced", shape, column bits) or ("grouped", shape, lanes per row of block 0)."""
    monkeypatch.setenv("MBAMG_VERBOSE", "1")
    capfd.readouterr()
    gpu_hierarchy(s, **kw).close()
    out = {}
    for line in capfd.readouterr().err.splitlines():
        m = re.search(r"level (\d+): sliced, shape (\d), (\d+)-bit columns", line)
        if m:
            out[int(m[1])] = ("sliced", int(m[2]), int(m[3]))
        m = re.search(r"level (\d+) block 0: .* (\d+) lanes per row, .* shape (\d)", line)
        if m:
            out[int(m[1])] = ("grouped", int(m[3]), int(m[2]))
    log(f"  {out}")
    return out


def _2d(n=23):
    return make_system(n, 2, 0.7, seed=3, kappa="lognormal", blk1_scale=2.0, a10_scale=0.5)


@pytest.mark.parametrize("split", ["1", "2", "16"])
@pytest.mark.parametrize("d", [1, 2, 3])
def test_16_bit_columns(d, split, capfd, monkeypatch):
    monkeypatch.setenv("MBAMG_ROWS_FORM", "sliced")
    monkeypatch.setenv("MBAMG_SLICE_SPLIT", split)
    s = _2d() if d == 3 else leading_components(_2d(), d)
    for ask in ("0", "1"):
        monkeypatch.setenv("MBAMG_COL16", ask)
        got = _layout(s, capfd, monkeypatch, max_coarse=60)
        bits = 16 if ask == "1" and split == "1" else 32
        assert len(got) >= 2 and all(v[0] == "sliced" and v[2] == bits for v in got.values())
    monkeypatch.setenv("MBAMG_COL16", "1")
    got = _layout(s, capfd, monkeypatch, max_coarse=60, smoother=1)
    assert got and all(v[2] == 32 for v in got.values())


def test_spread_columns_keep_32_bits(capfd, monkeypatch):
    monkeypatch.setenv("MBAMG_ROWS_FORM", "sliced")
    monkeypatch.setenv("MBAMG_COL16", "1")
    s = leading_components(make_system(400, 2, 0.7, seed=3), 1)
    assert _layout(s, capfd, monkeypatch, max_coarse=60)[0] == ("sliced", 0, 16)
    p = np.random.default_rng(3).permutation(s.N)
    for row in s.blocks:
        for k, a in enumerate(row):
            m = a.to_scipy()[p][:, p].tocsr()
            m.sort_indices()
            row[k] = type(a)(s.N, s.N, m.indptr.astype(np.int32), m.indices.astype(np.int32),
                             m.data.reshape(-1, 1, 1))
    assert _layout(s, capfd, monkeypatch, max_coarse=60)[0] == ("sliced", 0, 32)


@pytest.mark.parametrize("layout", ["grouped", "sliced"])
@pytest.mark.parametrize("what,shape", [("none", 2), ("scaled-all", 1), ("scaled-last", 1), ("full-last", 0),
                                        ("full-coupling", 0)])
def test_block_shapes(what, shape, layout, capfd, monkeypatch):
    from test_gpu_shapes import _break
    if layout == "sliced":
        monkeypatch.setenv("MBAMG_ROWS_FORM", "sliced")
    s = make_system(10, 3, 1.0, seed=5, kappa="lognormal")
    if what != "none":
        s = _break(s, what)
    got = _layout(s, capfd, monkeypatch, max_coarse=60)
    assert len(got) >= 2 and all(v[0] == layout for v in got.values())
    assert got[0][1] == shape
    if what == "none":
        assert all(v[1] == shape for v in got.values())


@pytest.mark.parametrize("n,dim,layout", [(32, 3, "grouped"), (33, 3, "sliced"), (256, 2, "grouped"), (257, 2, "sliced")])
def test_finest_levels(n, dim, layout, capfd, monkeypatch):
    s = leading_components(make_system(n, dim, 0.5), 1)
    got = _layout(s, capfd, monkeypatch)
    assert got[0][0] == layout and all(v[0] == "grouped" for l, v in got.items() if l > 0)
