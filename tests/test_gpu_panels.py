"""The register panels of the factorization at the edges of their shapes, run
on an MI355X: L = 1 cubes whose top separator has n^2 rows, so that the blocks
of 64 pivots end ragged and the panels' heights pass every row-wave count (64
to 768 rows, the taller kernel above), with few fronts at the top and many at
the leaves.  The local solve is checked by its residual under the oracle's own
assembly, with the tall-panel test's tolerances (1e-10, complex64 1e-3)."""

import numpy as np
import pytest

from helm_inputs import omega_for_ppw, smooth_random_model
from oracle.discretization import Problem

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("mixed", 1e-3)])
@pytest.mark.parametrize("n", [8, 9, 11, 13, 14, 16, 19, 22, 23, 27, 28, 30])
def test_single_layer_residual(n, precision, tol):
    import paper_1801_08655_amd as pt
    p = 3
    h = 1.0 / (n - 1)
    m = smooth_random_model((n, n, n), 0.25, 1.5, 0.75, 1.25, n)
    om = omega_for_ppw(0.75, h, 10.0)
    s = pt.Solver(m, h, om, p, 1, precision=precision, pml_C=25.0)
    rng = np.random.default_rng(n)
    r = rng.standard_normal((3, n, n, n)) + 1j * rng.standard_normal((3, n, n, n))
    w = s.layer_solve(0, torch.from_numpy(r).cuda()).cpu().numpy()
    R = r.reshape(3, -1).T
    res = R - Problem(m, h, om, p, 25.0).operator() @ w.reshape(3, -1).T
    err = (np.linalg.norm(res, axis=0) / np.linalg.norm(R, axis=0)).max()
    print(n, precision, err)
    assert err <= tol
    s.close()
