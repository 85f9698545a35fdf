"""The coarsest inverse where a panel's update and the next panel's pivots share
a launch: sizes with a ragged last panel, a last unit of columns and rows that
is not full, and fewer rows than one wavefront; a matrix with equal candidates
in every column (the tie rule) against LAPACK's LU solve."""
import numpy as np
import pytest

from gpu_util import gpu_hierarchy, rel, torch_dev
from paper_2103_07537_amd.inputs import make_system

pytestmark = pytest.mark.gpu


# 6 unknowns per node in two dimensions: n = 54, 96, 150, 294, 726, 1536, 2646 = 6 m^2
@pytest.mark.parametrize("m", [3, 4, 5, 7, 11, 16, 21])
@pytest.mark.parametrize("equal", [False, True])
def test_coarsest_inverse_edges(m, equal):
    s = make_system(m, 2, 0.5, seed=m)
    if equal:   # magnitudes rounded to powers of two: ties among the candidates of a column
        for row in s.blocks:
            for a in row:
                a.vals[...] = np.sign(a.vals) * np.exp2(np.round(np.log2(np.maximum(np.abs(a.vals), 2.0 ** -20))))
    A = s.to_scipy().toarray()
    cond = np.linalg.cond(A)
    hg = gpu_hierarchy(s, max_coarse=10 ** 6)
    assert hg.num_levels() == 1
    r = np.random.default_rng(m).standard_normal(s.n_dofs)
    z = torch_dev(np.zeros(s.n_dofs))
    hg.vcycle(torch_dev(r), z)
    ref = np.linalg.solve(A, r)
    # both solutions carry errors of about the condition number times the unit roundoff
    # (growth included, a hundred times that is ample)
    assert rel(z.cpu().numpy(), ref) <= max(1e-13, 100 * cond * 2.0 ** -53)
