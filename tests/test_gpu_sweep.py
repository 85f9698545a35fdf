"""The Gauss-Seidel sub-solve in one launch (4 to 64 lanes per row, rows waiting
for their neighbours of earlier colours) against the oracle: every group size,
one and several sweeps of both kinds, per-aggregate damping, blocks of 3 x 3 and
4 x 4, FP64 and FP32; the same cycle colour by colour (as timed launches are
enqueued) bit for bit; and a captured V-cycle replayed with other inputs and
eager cycles in between."""
import numpy as np
import pytest

from gpu_util import assert_close, gpu_hierarchy, log, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


def weights_fn(level, n_agg, F):
    k = np.arange(n_agg)
    return 0.1 + 0.6 * ((k * 37 + level) % 11) / 10.0, 0.5 + 0.5 * ((k * 13 + 3 * level) % 7) / 6.0


CASES = {
    "3d-11-lognormal": lambda: make_system(11, 3, 2.0, seed=5, kappa="lognormal", blk1_scale=1.7, a10_scale=0.6),
    "2d-37": lambda: make_system(37, 2, 0.7, seed=3, kappa="lognormal"),
}


# tolerances: the sums are the oracle's in another order, a few hundred terms (as in the
# other V-cycle parity tests): 1e-12 in FP64, 1e-5 in FP32
@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("group", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("sweeps", [(1, 1), (2, 1), (1, 2), (2, 3)])
@pytest.mark.parametrize("precision", [0, 1])
def test_every_group_size_matches_the_oracle(case, group, sweeps, precision, monkeypatch):
    from oracle import amg
    s = CASES[case]()
    kw = dict(max_coarse=60, bgs_sweeps=sweeps[0], inner_sweeps=sweeps[1])
    weighted = group in (8, 64)
    okw, gkw = dict(kw), dict(kw, precision=precision)
    if weighted:
        okw["weights"] = weights_fn
        gkw.update(weights=weights_fn, judge=0)
    ho = amg.setup(s.blocks, s.dofs, amg.Params(**okw), n_vec=s.n_vec)
    monkeypatch.setenv("MBAMG_SWEEP_GROUP", str(group))
    hg = gpu_hierarchy(s, **gkw)
    log(f"case={case} group={group} sweeps={sweeps} precision={precision} levels={hg.num_levels()}")
    assert hg.num_levels() == len(ho.levels) >= 3
    z = torch_dev(np.zeros(s.n_dofs))
    for seed in (1, 2):   # twice: the undamped buffers have changed places in between
        r = np.random.default_rng(seed).standard_normal(s.n_dofs)
        hg.vcycle(torch_dev(r), z)
        assert_close(z.cpu().numpy(), amg.vcycle(ho, r), 1e-12 if precision == 0 else 1e-5)
    # the same cycle with every colour launched by itself
    one = z.cpu().numpy().copy()
    hg.timing_enable(1)
    hg.vcycle(torch_dev(r), z)
    assert z.cpu().numpy().tobytes() == one.tobytes()
    hg.close()


@pytest.mark.parametrize("group", ["3", "128"])
def test_other_group_sizes_are_rejected(group, monkeypatch):
    from paper_2103_07537_amd import mbamg
    monkeypatch.setenv("MBAMG_SWEEP_GROUP", group)
    with pytest.raises(mbamg.MbamgError):
        gpu_hierarchy(make_system(12, 2, 0.5, seed=2), max_coarse=40)


@pytest.mark.parametrize("precision", [0, 1])
def test_captured_cycle_replays(precision):
    import torch
    s = CASES["3d-11-lognormal"]()
    hg = gpu_hierarchy(s, max_coarse=60, precision=precision)
    rng = np.random.default_rng(4)
    r, z, ze = (torch_dev(np.zeros(s.n_dofs)) for _ in range(3))
    r.copy_(torch_dev(rng.standard_normal(s.n_dofs)))
    hg.vcycle(r, z)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        hg.vcycle(r, z)
    for _ in range(4):
        r.copy_(torch_dev(rng.standard_normal(s.n_dofs)))
        hg.vcycle(r, ze)
        torch.cuda.synchronize()
        z.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, ze)
    hg.close()


def test_a_nan_in_the_input_ends_the_cycle():
    """A NaN whose bits are all ones is what an unwritten value looks like: it must come out as a NaN, and no
    wait may take it for a missing value."""
    import torch
    s = CASES["3d-11-lognormal"]()
    for precision in (0, 1):
        hg = gpu_hierarchy(s, max_coarse=60, precision=precision)
        r = np.random.default_rng(6).standard_normal(s.n_dofs)
        r.view(np.uint64)[[0, s.n_dofs // 2, s.n_dofs - 1]] = 0xFFFFFFFFFFFFFFFF
        z = torch_dev(np.zeros(s.n_dofs))
        hg.vcycle(torch_dev(r), z)
        torch.cuda.synchronize()
        assert torch.isnan(z).any()
        r = np.random.default_rng(7).standard_normal(s.n_dofs)   # and the next cycle is whole again
        hg.vcycle(torch_dev(r), z)
        assert torch.isfinite(z).all()
        hg.close()


# more than two blocks: the couplings (3 x 1, 1 x 3, 3 x 3, 1 x 1 blocks) are summed with the sweep
@pytest.mark.parametrize("split", ["3d-split4", "2d-split3"])
@pytest.mark.parametrize("group", [4, 16, 64])
@pytest.mark.parametrize("sweeps", [(1, 1), (2, 2)])
def test_more_than_two_blocks_with_every_group_size(split, group, sweeps, monkeypatch):
    from oracle import amg, nblock
    from paper_2103_07537_amd import mbamg
    from paper_2103_07537_amd.inputs import split_fields
    t = split_fields(make_system(11, 3, 0.6, seed=5, kappa="lognormal")) if split == "3d-split4" else \
        split_fields(make_system(25, 2, 0.5, seed=4), split_second=False)
    kw = dict(max_coarse=60, bgs_sweeps=sweeps[0], inner_sweeps=sweeps[1])
    ho = nblock.setup(t.blocks, t.dofs, amg.Params(**kw))
    monkeypatch.setenv("MBAMG_SWEEP_GROUP", str(group))
    hg = mbamg.Hierarchy(t.blocks, t.dofs, t.n_vec, **kw)
    assert hg.num_levels() == len(ho.levels) >= 3
    z, w = torch_dev(np.zeros(t.n_dofs)), torch_dev(np.zeros(t.n_dofs))
    for seed in (1, 2):
        r = np.random.default_rng(seed).standard_normal(t.n_dofs)
        hg.vcycle(torch_dev(r), z)
        assert_close(z.cpu().numpy(), nblock.vcycle(ho, r), 1e-12)
    hg.apply(torch_dev(r), w)
    ref = t.to_scipy() @ r
    assert np.max(np.abs(w.cpu().numpy() - ref)) <= 1e-13 * np.max(np.abs(ref))
    hg.close()
