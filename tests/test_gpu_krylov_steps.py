"""The Krylov passes with their sums finished by the last block, at sizes around
one block and one counter group (256 unknowns per block, 16 groups), and steps
enqueued ahead of the host: iteration counts and solutions against the oracle, and
bit for bit those of a solve that waits for every step (as timed solves do),
including caps on the iterations and restarts that end in the step ahead."""
import numpy as np
import pytest

from gpu_util import gpu_hierarchy, log, rel, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


# 2D grids of n x n nodes, 6 unknowns each: 1, 1, 16, 17, 18 and 61 blocks
@pytest.mark.parametrize("n", [5, 6, 26, 27, 28, 51])
@pytest.mark.parametrize("kw", [dict(), dict(restart=3), dict(restart=1, max_iters=7), dict(max_iters=5)],
                         ids=["30", "3", "1-cap7", "cap5"])
def test_steps_ahead_change_nothing(n, kw):
    from oracle import amg
    s = make_system(n, 2, 0.7, seed=3, kappa="lognormal")
    ho = amg.setup(s.blocks, s.dofs, amg.Params(max_coarse=60), n_vec=s.n_vec)
    for precision in (0, 1):
        h = gpu_hierarchy(s, max_coarse=60, precision=precision, **kw)
        out = []
        for mode in (0, 2, 0):
            h.timing_enable(mode)
            x = torch_dev(np.zeros(s.n_dofs))
            info = h.solve(torch_dev(s.b), x, rtol=1e-8)
            out.append((x.cpu().numpy(), info["iterations"], info["converged"]))
        for o in out[1:]:
            assert o[0].tobytes() == out[0][0].tobytes() and o[1:] == out[0][1:]
        if "max_iters" in kw:
            assert out[0][1] <= kw["max_iters"]
        else:
            xo, io = amg.gmres(ho, s.b, rtol=1e-8, restart=kw.get("restart", 30))
            log(f"n={n} {kw} precision={precision}: {out[0][1]} iterations, oracle {io.iterations}")
            # (restarted after 3 steps the largest system stalls, on both sides alike)
            assert out[0][2] == io.converged and abs(out[0][1] - io.iterations) <= 1
            if precision == 0 and io.converged and out[0][1] == io.iterations:
                assert rel(out[0][0], xo) <= 1e-8
        h.close()
