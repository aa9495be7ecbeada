"""Two-step smoothing in x tiles (rows of 4 KB and more) and passes of odd
degree that prolong inside their first pair (rows of 2 KB and more): each step
is formed as the single-step kernel forms it, so solves agree bitwise with
MG_OPT_NO_PAIR, cycle by cycle.  1024^3 double is the largest grid of the
tiles, 512^3 double and 1024^3 float the smallest of each type; degrees 2 to 5
reach every start of a pair (plain, from b, x_prev from b, prolonging) with
and without its first step written."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,degree", [(512, "fp64", 5), (1024, "mixed", 2), (1024, "mixed", 3),
                                           (1024, "mixed", 4), (1024, "mixed", 5), (1024, "fp64", 4),
                                           (512, "mixed", 5), (256, "fp64", 5)])
def test_pairs_on_long_rows_match_single_steps(n, prec, degree):
    import paper_2607_10983_amd as mg
    torch.manual_seed(n + degree)
    b = torch.randn((n, n, n), device="cuda", dtype=torch.float64)
    b -= b.mean()
    kw = dict(levels=n.bit_length() - 2, degree=degree, precision=prec)
    out = []
    for options in (mg._lib.MG_OPT_NO_PAIR, 0):
        m = mg.Multigrid(n, options=options, **kw)
        phi, info = m.solve(b, tol=1e-10, max_cycles=2, raise_on_error=False)
        out.append((phi, info.history))
        del m
    assert out[0][1] == out[1][1]
    assert torch.equal(out[0][0], out[1][0])
