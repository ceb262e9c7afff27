"""Solves at the edges of the dot products' column tiles (1, 2, 4, 8, 16 and 32
columns), run on an MI355X: a wrong or mixed-up dot product breaks the Arnoldi
basis of its column, so that column misses the oracle's direct solve.  The
bound is the batched solve's (1e-9)."""

import numpy as np
import pytest

from helm_inputs import omega_for_ppw, smooth_random_model
from oracle.direct import SparseLU, relative_error
from oracle.discretization import Problem, point_source_rhs

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33])
def test_solve_at_dot_tile_edges(k):
    import paper_1801_08655_amd as pt
    grid, p, L, alpha = (17, 15, 18), 3, 3, 2
    h = 1.0 / (max(grid) - 1)
    m = smooth_random_model(grid, 0.25, 2.0, 0.75, 1.25, 6)
    om = omega_for_ppw(0.75, h, 10.0)
    pb = Problem(m, h, om, p, 25.0)
    srcs = [(4 + (3 * i) % 9, 4 + (5 * i) % 7, 4 + (7 * i) % 10) for i in range(k)]
    ref = SparseLU(pb.operator()).solve(point_source_rhs(pb.shape, srcs, h))
    s = pt.Solver(m, h, om, p, L, precision="fp64", pml_C=25.0, pml_local=alpha)
    u = s.solve_points(srcs).cpu().numpy().reshape(k, -1).T
    assert relative_error(u, ref).max() <= 1e-9
    s.close()
