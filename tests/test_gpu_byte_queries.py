"""The byte model's queries take a const hierarchy and are host arithmetic: they
may be asked while another stream is being captured, and by several threads at
once, from the first call on."""
import threading

import numpy as np
import pytest

from gpu_util import gpu_hierarchy, log, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


def _system():
    return make_system(11, 3, 2.0, seed=5, kappa="lognormal")


def _all_bytes(h):
    return [h.vcycle_bytes()] + [b for l in range(h.num_levels()) for b in h.level_vcycle_bytes(l)]


def test_queries_during_a_capture():
    import torch
    s = _system()
    h = gpu_hierarchy(s, max_coarse=60)
    r, z, ze = (torch_dev(np.zeros(s.n_dofs)) for _ in range(3))
    r.copy_(torch_dev(np.random.default_rng(3).standard_normal(s.n_dofs)))
    h.vcycle(r, ze)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        h.vcycle(r, z)
        during = _all_bytes(h)
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(z, ze)
    assert during == _all_bytes(h) and min(during) >= 0.0 and during[0] > 0.0
    h.close()


def test_queries_from_several_threads():
    s = _system()
    ref = gpu_hierarchy(s, max_coarse=60)
    expected = _all_bytes(ref)
    ref.close()
    h = gpu_hierarchy(s, max_coarse=60)
    start, got = threading.Barrier(8), [None] * 8

    def ask(k):
        start.wait()
        got[k] = _all_bytes(h)

    threads = [threading.Thread(target=ask, args=(k,)) for k in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    log(f"  {expected[0]:.0f} B per V-cycle")
    assert got == [expected] * 8
    h.close()
