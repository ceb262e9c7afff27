"""The allocation-free local solve at its limit, run on an MI355X: the widest
batch that fits the array when its split-K partials are counted at chunks of at
least 256 rows.  The launches' finer chunks need more than that, so the columns
go in two passes; one more column is refused.  Against the allocating entry
point with the existing test's bound (1e-12)."""

import numpy as np
import pytest

from helm_inputs import omega_for_ppw, smooth_random_model
from oracle.direct import relative_error

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


# one layer of 60 x 60 x 22 in complex128: 28 columns at most, 25 in one pass;
# 68 x 68 x 30: 16 and 15
@pytest.mark.parametrize("grid,k_max", [((60, 60, 22), 28), ((68, 68, 30), 16)])
def test_widest_accepted_batch(grid, k_max):
    import paper_1801_08655_amd as pt
    nx, ny, nz = grid
    h = 1.0 / (nx - 1)
    m = smooth_random_model(grid, 0.25, 2.0, 0.75, 1.25, 3)
    om = omega_for_ppw(0.75, h, 10.0)
    s = pt.Solver(m, h, om, 3, 1, precision="fp64", pml_C=25.0)

    def call(r, w):
        return pt.lib().helm_layer_solve_noalloc_dev(s._h, 0, r.shape[0], r.data_ptr(),
                                                     w.data_ptr())

    g = torch.Generator(device="cuda")
    g.manual_seed(k_max)
    r = torch.randn((k_max + 1, nz, ny, nx), dtype=torch.complex128, device="cuda", generator=g)
    w = torch.empty_like(r)
    torch.cuda.synchronize()
    assert call(r, w) == pt.HELM_ENOMEM
    for k in (k_max, k_max - 1):
        w.zero_()
        torch.cuda.synchronize()
        assert call(r[:k], w[:k]) == pt.HELM_OK
        a = w[:k].cpu().numpy().reshape(k, -1).T
        b = s.layer_solve(0, r[:k]).cpu().numpy().reshape(k, -1).T
        assert relative_error(a, b).max() <= 1e-12
        assert np.all(w[k:].cpu().numpy() == 0)
    s.close()
