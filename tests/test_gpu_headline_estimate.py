"""The mixed-precision headline workload (200^3, L = 20, 64 sources, the
refinement options of bench.py without measured tiles), run on an MI355X against
the complex128 path: every column stops on its estimate within the target, and
where a column's true error matters (above a tenth of the target) its estimate
is at least half of it, the bound that the smaller workloads' estimates are held
to."""

import numpy as np
import pytest

from helm_inputs import workload

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


def test_layered_200_estimates_cover_the_errors():
    import paper_1801_08655_amd as pt
    wl = workload("layered-200")
    m = wl.m()
    srcs = wl.point_sources(64)
    kw = dict(pml_local=wl.pml_local, pml_C=wl.pml_C)
    s = pt.Solver(m, wl.h, wl.omega, wl.pml, wl.n_layers, precision="mixed", ir_tol=1e-10,
                  inner_tol=5e-4, inner_tol_refine=2e-4, err_target=1e-6, ir_max_steps=4, **kw)
    u, info = s.solve_points(srcs, info=True)
    s.close()
    s = pt.Solver(m, wl.h, wl.omega, wl.pml, wl.n_layers, precision="fp64", gmres_tol=1e-10,
                  max_rhs=32, **kw)
    v = s.solve_points(srcs)
    s.close()
    err = np.array([(torch.linalg.vector_norm(u[c] - v[c]) /
                     torch.linalg.vector_norm(v[c])).item() for c in range(64)])
    est = np.array(info["rhs_est_error"])
    print("errors: max", err.max(), "median", np.median(err), "estimates: max", est.max())
    assert info["ir_steps"] < 4 and est.max() <= 1e-6
    assert err.max() <= 1e-6
    big = err > 1e-7
    assert np.all(est[big] >= 0.5 * err[big])
