"""The 19-point step that prolongs on the fly (float rows of 64^3 to 256^3,
double of 64^3 and 128^3): the rounding of the separate prolongation and step,
so solves agree bitwise with MG_OPT_NO_PAIR.  Degree 1 keeps no x_0, degrees 2
and 3 hand it to a single step or a pair; Jacobi sweeps need none."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(64, "mixed"), (128, "mixed"), (256, "mixed"), (64, "fp64"), (128, "fp64")])
@pytest.mark.parametrize("smoother,degree", [("chebyshev", 1), ("chebyshev", 2), ("chebyshev", 3), ("chebyshev", 4),
                                             ("jacobi", 1), ("jacobi", 2)])
def test_matches_prolongation_and_step(n, prec, smoother, degree):
    import paper_2607_10983_amd as mg
    torch.manual_seed(n + degree)
    g = torch.arange(n, device="cuda", dtype=torch.float64) * (6.283185307179586 / n)
    psi = 2e-3 * torch.sin(g)[:, None, None] * torch.sin(2 * g)[None, :, None] * torch.cos(g)[None, None, :]
    b = torch.randn((n, n, n), device="cuda", dtype=torch.float64)
    b -= b.mean()
    kw = dict(levels=n.bit_length() - 2, psi=psi, precision=prec, smoother=smoother, degree=degree, sweeps=degree)
    out = []
    for options in (mg._lib.MG_OPT_NO_PAIR, 0):
        m = mg.Multigrid(n, options=options, **kw)
        phi, info = m.solve(b, tol=0.0, max_cycles=3, raise_on_error=False)
        out.append((phi, info.history))
    assert out[0][1] == out[1][1]
    assert torch.equal(out[0][0], out[1][0])
