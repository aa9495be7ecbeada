"""Reverse mode of the geometry in tiles of 32 x 8 points, at grids smaller than
a tile, of one tile and of many, against the geometry itself: <Cbar, dC> +
<sbar, dsqrtg> along a direction equals <psibar, direction>; and a psibar that
replaces an input."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


def field(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((n, n, n), generator=g, device="cuda", dtype=torch.float64)


def smooth(n, seed):
    f = field(n, seed)
    for d in range(3):
        for _ in range(2):
            f = 0.25 * torch.roll(f, 1, d) + 0.5 * f + 0.25 * torch.roll(f, -1, d)
    return f


@pytest.mark.parametrize("n", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("with_sbar", [True, False])
def test_directional_derivative(n, with_sbar):
    import paper_2607_10983_amd as mg
    psi = 0.02 * smooth(n, 1) / n ** 2
    v = smooth(n, 2) / n ** 2
    Cbar = torch.stack([field(n, 3 + c) for c in range(6)])
    sbar = field(n, 9) if with_sbar else None
    bar = mg.geometry_bwd(psi, Cbar, sbar)
    # J changes by 5e-5 along the difference: its third-order term is below 1e-8
    # of the derivative, the rounding of C (1e-16 / 1e-5) below 1e-10
    eps = 1e-5
    (Cp, sp), (Cm, sm) = mg.geometry(psi + eps * v), mg.geometry(psi - eps * v)
    want = float((Cbar * (Cp - Cm)).sum() / (2 * eps))
    scale = float((Cbar * (Cp - Cm)).abs().sum() / (2 * eps))
    if with_sbar:
        want += float((sbar * (sp - sm)).sum() / (2 * eps))
        scale += float((sbar * (sp - sm)).abs().sum() / (2 * eps))
    assert abs(float((bar * v).sum()) - want) <= 1e-8 * scale


@pytest.mark.parametrize("n", [16, 64])
@pytest.mark.parametrize("entry", ["mg_geometry_bwd", "mg_geometry_bwd_noalloc"])
def test_result_may_replace_an_input(n, entry):
    import paper_2607_10983_amd as mg
    from paper_2607_10983_amd import _lib
    psi, Cbar, sbar = 0.02 * smooth(n, 1) / n ** 2, torch.stack([field(n, 3 + c) for c in range(6)]), field(n, 9)
    want = mg.geometry_bwd(psi, Cbar, sbar)
    for which in range(3):
        a = [psi.clone(), Cbar.clone(), sbar.clone()]
        out = a[which][2] if which == 1 else a[which]
        p = [ctypes.c_void_p(t.data_ptr()) for t in a]
        st = getattr(_lib.load(), entry)(n, 1.0 / n, *p, ctypes.c_void_p(out.data_ptr()),
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == _lib.MG_OK
        torch.cuda.synchronize()
        assert torch.equal(out, want)
