"""HELM_FLAG_GEMM_4M and HELM_FLAG_FACTOR_4M, run on an MI355X: both are accepted
and change nothing, since complex64 products are always formed from four real
ones.  Widths from 5 columns on take the matrix-core tile (fewer the vector
kernels): bit for bit the same local solves in both precisions, the narrowest
widths also against SuperLU on the oracle's H^l (2e-5, the bound of the other
complex64 local solves)."""

import numpy as np
import pytest

from helm_inputs import omega_for_ppw, smooth_random_model
from oracle.direct import SparseLU, relative_error
from oracle.discretization import Problem, local_operator

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision,tol", [("mixed", 2e-5), ("fp64", 1e-11)])
def test_flags_change_nothing(precision, tol):
    import paper_1801_08655_amd as pt
    nx, ny, nz, p, L, alpha = 23, 18, 29, 4, 3, 3
    h = 1.0 / (nz - 1)
    m = smooth_random_model((nx, ny, nz), 0.25, 2.0, 0.75, 1.25, 6)
    om = omega_for_ppw(0.75, h, 10.0)
    lu = SparseLU(local_operator(Problem(m, h, om, p, 25.0), L, alpha, 1))
    flag = pt._lib.HELM_FLAG_GEMM_4M, pt._lib.HELM_FLAG_FACTOR_4M
    s = [pt.Solver(m, h, om, p, L, precision=precision, pml_C=25.0, pml_local=alpha, flags=f)
         for f in (0, flag[0], flag[1], flag[0] | flag[1])]
    lo, hi = s[0].layer_info(1)[2:]
    rng = np.random.default_rng(5)
    r = rng.standard_normal((33, hi - lo + 1, ny, nx)) * (1 + 1j)
    r.imag = rng.standard_normal(r.shape)
    rt = torch.from_numpy(r).cuda()
    for k in (5, 6, 16, 17, 33):
        w = [x.layer_solve(1, rt[:k]) for x in s]
        assert all(torch.equal(w[0], x) for x in w[1:]), k
        if k <= 6:
            err = relative_error(w[0].cpu().numpy().reshape(k, -1).T,
                                 lu.solve(r[:k].reshape(k, -1).T))
            print(precision, "k", k, "rel err", err.max())
            assert err.max() <= tol
    for x in s:
        x.close()
