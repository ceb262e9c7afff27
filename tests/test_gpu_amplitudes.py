"""Mixed precision far from amplitude 1, run on an MI355X.  Every entry point is
linear per column, so a column times a power of two has the answer times that
power: exactly so in FP64 arithmetic, and in complex64 as long as nothing leaves
the range in which its products are formed exactly (about 2^-110 to 2^127),
which the entry points see to by scaling such columns.  Widths on both sides of
the matrix-core tile's (5 and more columns); one column of an ordinary amplitude
sits between the others.

Tolerance: a power of two commutes with every rounding, so the scaled answer is
the unscaled one to the last bit of complex64 data, up to where a column alone
is scaled (a different power of two, the same bits): 1e-12 of the column."""

import numpy as np
import pytest

from helm_inputs import omega_for_ppw, smooth_random_model

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")

EXPONENTS = (-300, -126, -112, -104, -60, 60, 110, 127, 300)


@pytest.fixture(scope="module")
def solver():
    import paper_1801_08655_amd as pt
    n, p, L = 24, 4, 3
    h = 1.0 / (n - 1)
    m = smooth_random_model((n, n, n), 0.25, 2.0, 0.75, 1.25, 5)
    s = pt.Solver(m, h, omega_for_ppw(0.75, h, 8.0), p, L, precision="mixed", ir_tol=1e-10)
    yield s
    s.close()


def _check(got, want, scale):
    """Columns of got (k, ...) against scale[c] times those of want."""
    for c, s in enumerate(scale):
        a = got[c].ravel() * (1.0 / s)
        d = torch.linalg.vector_norm(a - want[c].ravel())
        assert d <= 1e-12 * torch.linalg.vector_norm(want[c].ravel()), (c, s)


def _scales(k, e):
    s = np.full(k, 2.0 ** e)
    s[k // 2] = 1.0
    return s


@pytest.mark.parametrize("k", [2, 7])
@pytest.mark.parametrize("e", EXPONENTS)
def test_local_solves(solver, k, e):
    lo, hi = solver.layer_info(1)[2:]
    nx, ny, _ = solver.n
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    r = torch.randn((k, hi - lo + 1, ny, nx), dtype=torch.complex128, device="cuda", generator=g)
    sc = _scales(k, e)
    rs = r * torch.from_numpy(sc).cuda().reshape(-1, 1, 1, 1)
    for solve in (solver.layer_solve, solver.layer_solve_noalloc):
        want = solve(1, r)
        keep = rs.clone()
        _check(solve(1, rs), want, sc)
        assert torch.equal(rs, keep)
    # in place
    w = rs.clone()
    solver.layer_solve_noalloc(1, w, w)
    _check(w, want, sc)


@pytest.mark.parametrize("e", EXPONENTS)
def test_interface_operators(solver, e):
    k = 7
    nx, ny, nz = solver.n
    vp = (solver.n_layers - 1) * 2 * nx * ny * k
    sc = _scales(k, e)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    for op in range(5):
        size = (k * nz * ny * nx) if op >= 3 else (vp if op == 2 else 2 * vp)
        x = torch.randn(size, dtype=torch.complex128, device="cuda", generator=g)
        st = torch.from_numpy(sc).cuda()
        xs = (x.reshape(k, -1) * st[:, None] if op >= 3 else x.reshape(-1, k) * st).reshape(-1)
        want = solver.polarized_op(op, x, k).reshape(-1, k).T
        _check(solver.polarized_op(op, xs, k).reshape(-1, k).T, want, sc)


@pytest.mark.parametrize("k", [2, 7])
@pytest.mark.parametrize("e", (-140, -110, -80, 80, 127, 140))
def test_refined_solves(solver, k, e):
    """The refinement works on residuals down to 1e-10 of the source.  Its steps
    and answers are those of amplitude 1."""
    nodes = [(6 + c, 17 - c, 7 + c) for c in range(k)]
    want, a = solver.solve_points(nodes, np.ones(k), info=True)
    sc = _scales(k, e)
    got, b = solver.solve_points(nodes, sc, info=True)
    assert b["rhs_ir_steps"] == a["rhs_ir_steps"]
    _check(got, want, sc)


@pytest.mark.parametrize("k", [2, 7])
def test_tiny_tails_in_an_ordinary_column(solver, k):
    """Values far below the column's own size do not have the column scaled, in
    place or not: bit for bit the answer of any ordinary call's path."""
    lo, hi = solver.layer_info(1)[2:]
    nx, ny, _ = solver.n
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    r = torch.randn((k, hi - lo + 1, ny, nx), dtype=torch.complex128, device="cuda", generator=g)
    z = r.clone()
    z[:, 0] = 0
    r[:, 0] = 1e-30   # (vanishes beside the rest in complex64)
    want = solver.layer_solve(1, z)
    got = solver.layer_solve(1, r)
    d = torch.linalg.vector_norm(got - want)
    assert d <= 1e-12 * torch.linalg.vector_norm(want)
    w = r.clone()
    assert torch.equal(solver.layer_solve_noalloc(1, w, w), got)
