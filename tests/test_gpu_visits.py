"""Level visits of the 32^3 level in a double hierarchy: the point formulas of
the separate kernels, so solves agree bitwise with MG_OPT_NO_VISIT, cycle by
cycle.  Degrees 1 to 4 are the halo widths of the tiles; 5 runs unfused."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels", [(32, 2), (32, 4), (64, 3), (128, 6)])
@pytest.mark.parametrize("degree", [1, 2, 3, 4, 5])
def test_double_visits_match_separate_kernels(n, levels, degree):
    import paper_2607_10983_amd as mg
    torch.manual_seed(n + degree)
    b = torch.randn((n, n, n), device="cuda", dtype=torch.float64)
    b -= b.mean()
    out = []
    for options in (mg._lib.MG_OPT_NO_VISIT, 0):
        m = mg.Multigrid(n, levels=levels, degree=degree, precision="fp64", options=options)
        phi, info = m.solve(b, tol=0.0, max_cycles=3, raise_on_error=False)
        out.append((phi, info.history))
    assert out[0][1] == out[1][1]
    assert torch.equal(out[0][0], out[1][0])
