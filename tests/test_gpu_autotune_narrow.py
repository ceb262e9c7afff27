"""Measured tile choices for batches of up to 4 columns, run on an MI355X: the
vector path (one launch per depth and pass) against matrix-core tiles whose pass
also takes gather and reduction launches.  Every depth's choice is the quickest
of the measured passes, lists whose launches differ are measured on their own,
and the solution is that of the default choices (complex128, 1e-12: the widths
change the order of sums only)."""

import pytest

from helm_inputs import omega_for_ppw, smooth_random_model
from oracle.direct import relative_error

pytestmark = [pytest.mark.gpu,
              pytest.mark.filterwarnings("ignore::DeprecationWarning")]

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [1, 3, 4])
def test_narrow_choices(k):
    import paper_1801_08655_amd as pt
    n, p, L = 40, 5, 4
    h = 1.0 / (n - 1)
    m = smooth_random_model((n, n, n), 0.25, 2.0, 0.75, 1.25, 2)
    om = omega_for_ppw(0.75, h, 8.0)
    nodes = [(8 + 3 * c, 9, 7 + 2 * c) for c in range(k)]
    u = {}
    for flags in (0, pt._lib.HELM_FLAG_AUTOTUNE):
        s = pt.Solver(m, h, om, p, L, precision="fp64", flags=flags)
        u[flags] = s.solve_points(nodes).cpu().numpy().reshape(k, -1).T
        if flags:
            recs = [c for c in s.tile_choices() if c["k"] == k]
        s.close()
    assert relative_error(u[pt._lib.HELM_FLAG_AUTOTUNE], u[0]).max() <= 1e-12
    kinds = (1, 16)
    for c in recs:
        for bn, t in ((c["fwd_bn"], c["t_fwd_us"]), (c["bwd_bn"], c["t_bwd_us"])):
            tried = {b: t[i] for i, b in enumerate(kinds) if t[i] > 0}
            if tried:
                assert tried.get(bn, 0) == min(tried.values())
        if c["fwd_elems"] > 0:
            assert c["t_fwd_us"][0] > 0 and c["t_fwd_us"][1] > 0
    # a time that two records share was measured once for both: their work is
    # alike (a bucket's mean sizes lie within a factor 2^(1/4), so the product
    # of two within 2^(1/2))
    seen = {}
    for c in recs:
        if c["fwd_elems"] > 0:
            seen.setdefault((c["t_fwd_us"][0], c["t_fwd_us"][1]), []).append(c["fwd_elems"])
    for e in seen.values():
        assert max(e) <= 1.5 * min(e), e
