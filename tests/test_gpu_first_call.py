"""Device memory that a new handle's first solve takes, run on an MI355X: up to 4
columns run on the vector kernels, which have no split-K partial products, so no
room for them is taken (measured tile choices may pick the matrix-core tile and
take it).  Wider batches after narrower ones still get what they need."""

import pytest

from helm_inputs import omega_for_ppw, smooth_random_model

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


def test_no_partial_products_up_to_4_columns():
    import paper_1801_08655_amd as pt
    n, p, L = 100, 10, 4
    h = 1.0 / (n - 1)
    m = smooth_random_model((n, n, n), 0.25, 2.0, 0.75, 1.25, 2)
    om = omega_for_ppw(0.75, h, 8.0)
    took, w = {}, {}
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    r = None
    for flags in (0, pt._lib.HELM_FLAG_AUTOTUNE):
        s = pt.Solver(m, h, om, p, L, precision="fp64", flags=flags)
        if r is None:
            lo, hi = s.layer_info(1)[2:]
            r = torch.randn((9, hi - lo + 1, n, n), dtype=torch.complex128, device="cuda",
                            generator=g)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        out = torch.empty_like(r)   # (torch's pool may grow for the results)
        del out
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        a = s.layer_solve(1, r[:4])
        torch.cuda.synchronize()
        took[flags] = free - torch.cuda.mem_get_info()[0]
        b = s.layer_solve(1, r)
        w[flags] = (a, b)
        s.close()
    print("first solve took", took)
    # the partials of 4 columns at this size: several MB
    assert took[0] <= took[pt._lib.HELM_FLAG_AUTOTUNE] - (1 << 20)
    for x, y in zip(*w.values()):
        assert torch.linalg.vector_norm(x - y) <= 1e-12 * torch.linalg.vector_norm(y)
    a, b = w[0]
    assert torch.linalg.vector_norm(a - b[:4]) <= 1e-11 * torch.linalg.vector_norm(a)
