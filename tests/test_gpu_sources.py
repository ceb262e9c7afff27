"""The sweep solves' right-hand sides and read-outs in one launch each, where
the planes of a layer's two sides meet (layers of one and two bulk planes: the
top and bottom sources share planes), run on an MI355X: P (M x) and U x against
the oracle's unfused operators, with the bound of the existing operator test
(1e-10)."""

import numpy as np
import pytest

from helm_inputs import omega_for_ppw, smooth_random_model
from oracle.direct import relative_error
from oracle.discretization import Problem
from oracle.polarized import PolarizedTraces

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [1, 5])
@pytest.mark.parametrize("planes,L", [(4, 4), (7, 4)])
def test_thin_layers(planes, L, k):
    import paper_1801_08655_amd as pt
    nx, ny, p, alpha = 13, 11, 3, 2
    nz = planes + 2 * p
    h = 1.0 / (nx - 1)
    m = smooth_random_model((nx, ny, nz), 0.25, 2.0, 0.75, 1.25, 4)
    om = omega_for_ppw(0.75, h, 10.0)
    s = pt.Solver(m, h, om, p, L, precision="fp64", pml_C=25.0, pml_local=alpha)
    cpu = PolarizedTraces(Problem(m, h, om, p, 25.0), L, alpha)
    rng = np.random.default_rng(k)
    shape = cpu.zero_pairs().shape
    xd, xu = ([rng.standard_normal(shape) + 1j * rng.standard_normal(shape) for _ in range(k)]
              for _ in range(2))
    flat = lambda x: np.stack(x, axis=-1).ravel()  # noqa: E731
    gx = torch.from_numpy(np.concatenate([flat(xd), flat(xu)])).cuda()
    got = s.polarized_op(1, gx, k).cpu().numpy()
    ref = [cpu.precondition(*cpu.apply_M(a, b)) for a, b in zip(xd, xu)]
    ref = np.concatenate([flat([r[0] for r in ref]), flat([r[1] for r in ref])])
    assert relative_error(got, ref)[0] <= 1e-10
    got = s.polarized_op(2, torch.from_numpy(flat(xu)).cuda(), k).cpu().numpy()
    assert relative_error(got, flat([cpu.U_op(x) for x in xu]))[0] <= 1e-10
    s.close()
