"""Work counts of a profiled factorization, run on an MI355X, against an
independent nested-dissection plan: the sweep's bytes are the entries of the
tiles that it does not skip (the mirrored ones above the diagonal of the boundary
block among them), read and written, and the pivot rows and columns."""

import pytest

import test_library_cpu as tlc
from helm_inputs import omega_for_ppw, smooth_random_model

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


def _sweep_bytes(s, b, elem, nb=64, T=64):
    n, total = s + b, 0.0
    for k in range(0, s, nb):
        w = min(nb, s - k)
        for i0 in range(0, n, T):
            for j0 in range(0, n, T):
                pivot = any(x >= k and x + T <= k + w for x in (i0, j0))
                done = i0 + T <= k and j0 >= s
                mirrored = i0 >= s and j0 >= i0 + T
                if not (pivot or done or mirrored):
                    total += 2.0 * min(T, n - i0) * min(T, n - j0)
        total += 2.0 * n * w
    return total * elem


@pytest.mark.parametrize("precision,elem", [("fp64", 16), ("mixed", 8)])
def test_sweep_bytes(precision, elem):
    import paper_1801_08655_amd as pt
    n, p, L, alpha = 40, 5, 3, 4
    h = 1.0 / (n - 1)
    m = smooth_random_model((n, n, n), 0.25, 2.0, 0.75, 1.25, 2)
    s = pt.Solver(m, h, omega_for_ppw(0.75, h, 8.0), p, L, precision=precision,
                  pml_local=alpha, flags=pt._lib.HELM_FLAG_PROFILE)
    got = s.kernel_stats()["factor_sweep_gemm"]["bytes"]
    s.close()
    want = sum(_sweep_bytes(a, b, elem) for t in tlc._layer_planes(n, p, L, alpha)
               for a, b in tlc._nd_count(n, n, t, 64))
    assert got == pytest.approx(want, rel=1e-12)
