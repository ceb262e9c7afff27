"""The complex64 GEMM tile on the bf16 matrix cores (floats split exactly into
three bf16 numbers), run on an MI355X: local solves at the batch widths where
its column tiles end (16, 32 and 64 columns, one past each, two tiles), on a
grid whose fronts end inside row tiles and K steps, each column against
SuperLU on the oracle's H^l.

Tolerance: the one the vector kernels' complex64 local solves are held to
(2e-5; they measure 1e-6): the split products are at least as accurate as
FP32 ones."""

import numpy as np
import pytest

from helm_inputs import omega_for_ppw, smooth_random_model
from oracle.direct import SparseLU, relative_error
from oracle.discretization import Problem, local_operator

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def layer():
    import paper_1801_08655_amd as pt
    nx, ny, nz, p, L, alpha = 23, 18, 29, 4, 3, 3
    h = 1.0 / (nz - 1)
    m = smooth_random_model((nx, ny, nz), 0.25, 2.0, 0.75, 1.25, 6)
    om = omega_for_ppw(0.75, h, 10.0)
    s = pt.Solver(m, h, om, p, L, precision="mixed", pml_C=25.0, pml_local=alpha)
    lu = SparseLU(local_operator(Problem(m, h, om, p, 25.0), L, alpha, 1))
    lo, hi = s.layer_info(1)[2:]
    yield s, lu, (hi - lo + 1, ny, nx)
    s.close()


@pytest.mark.parametrize("k", [3, 15, 16, 17, 31, 33, 47, 64, 65, 129])
def test_local_solve_at_column_tile_edges(layer, k):
    s, lu, shape = layer
    rng = np.random.default_rng(k)
    r = rng.standard_normal((k,) + shape) + 1j * rng.standard_normal((k,) + shape)
    w = s.layer_solve(1, torch.from_numpy(r).cuda()).cpu().numpy()
    err = relative_error(w.reshape(k, -1).T, lu.solve(r.reshape(k, -1).T))
    print("k", k, "rel err", err.max())
    assert err.max() <= 2e-5
