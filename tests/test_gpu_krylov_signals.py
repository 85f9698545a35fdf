"""The Krylov passes' partial sums are their own signals (a value that is not there
yet is a NaN of all ones): sums that are that NaN must not be taken for missing ones,
and solves on 1 to many workgroups and of several restarts repeat bit for bit, with
sums of every kind of pass in between."""
import time

import numpy as np
import pytest

from gpu_util import gpu_hierarchy, log, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


def test_a_right_hand_side_of_all_ones_bits_ends():
    import torch
    s = make_system(24, 2, 0.5, seed=2)
    h = gpu_hierarchy(s, max_iters=6)
    b = s.b.copy()
    b.view(np.uint64)[::3] = 0xFFFFFFFFFFFFFFFF
    x = torch_dev(np.zeros(s.n_dofs))
    t = time.perf_counter()
    info = h.solve(torch_dev(b), x)
    took = time.perf_counter() - t
    log(f"  {1e3 * took:.1f} ms")
    assert not info["converged"] and took < 0.5   # a wait for one sum alone would take a second
    x.zero_()
    h2 = gpu_hierarchy(s)
    y = torch_dev(np.zeros(s.n_dofs))
    i1, i2 = h2.solve(torch_dev(s.b), y), None
    h.close()
    assert i1["converged"] and torch.isfinite(y).all()
    h2.close()


@pytest.mark.parametrize("n,dim", [(5, 2), (9, 2), (33, 2), (17, 3), (100, 2)])
@pytest.mark.parametrize("precision", [0, 1])
def test_solves_repeat_bit_for_bit(n, dim, precision):
    import torch
    s = make_system(n, dim, 0.5, seed=3, kappa="lognormal")
    h = gpu_hierarchy(s, max_coarse=60, precision=precision, restart=7)
    b, first = torch_dev(s.b), None
    for k in range(6):
        x = torch.zeros_like(b)
        info = h.solve(b, x)
        assert info["converged"]
        h.probe(5, 77)
        first = x if first is None else first
        assert torch.equal(x, first)
    A = s.to_scipy()
    assert np.linalg.norm(s.b - A @ first.cpu().numpy()) <= 1e-8 * np.linalg.norm(s.b) * (1 + 1e-6)
    h.close()
