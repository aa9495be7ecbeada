"""Residual and full weighting of the 19-point operator in one pass (rows of up
to 1 KB: float 64^3 to 256^3, double 64^3 and 128^3) and in two (256^3 double),
against the operator applied in double and a full weighting by shifts."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def full_weighting(r):
    for d in range(3):
        r = 0.25 * torch.roll(r, 1, d) + 0.5 * r + 0.25 * torch.roll(r, -1, d)
    return r[::2, ::2, ::2]


@pytest.mark.parametrize("n,prec", [(64, "mixed"), (128, "mixed"), (256, "mixed"), (64, "fp64"), (128, "fp64"),
                                    (256, "fp64")])
def test_residual_restrict(n, prec):
    import paper_2607_10983_amd as mg
    torch.manual_seed(n)
    g = torch.arange(n, device="cuda", dtype=torch.float64) * (6.283185307179586 / n)
    psi = 2e-3 * torch.sin(g)[:, None, None] * torch.sin(2 * g)[None, :, None] * torch.cos(g)[None, None, :]
    C = mg.geometry(psi)[0]
    x = torch.randn((n, n, n), device="cuda", dtype=torch.float64)
    b = torch.randn((n, n, n), device="cuda", dtype=torch.float64) * n * n
    if prec == "mixed":
        C, x, b = (t.float().double() for t in (C, x, b))
    levels = n.bit_length() - 2
    ref = mg.Multigrid(n, levels=levels, coeff=C, precision="fp64")
    expect = full_weighting(b - ref.apply(x))
    m = mg.Multigrid(n, levels=levels, coeff=C, precision=prec)
    out = m.inner_step("residual_restrict", 0, x=x, b=b)
    # 19 products and 27 weights: the bars of a single pass in each precision
    err = float((out - expect).abs().max() / expect.abs().max())
    assert err <= (5e-6 if prec == "mixed" else 1e-12), err
