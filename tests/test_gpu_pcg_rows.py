"""Conjugate-gradient passes on rows (the seven-point operator from 64^3): the
tiles of each row length (whole rows at 64 and 128, several tiles from 256),
both hierarchy types, the first iteration and a restart."""
import numpy as np
import pytest
import torch

from oracle import mg_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(64, "fp64"), (128, "fp64")])
def test_iterates_match_oracle(n, prec):
    import paper_2607_10983_amd as mg
    rng = np.random.default_rng(n)
    b = rng.standard_normal((n, n, n))
    phi0 = rng.standard_normal((n, n, n)) * 1e-3
    levels = n.bit_length() - 2
    H = O.build_hierarchy(n, levels)
    ref = O.solve_pcg(H, b, phi0=phi0, tol=0.0, max_iter=4)
    m = mg.Multigrid(n, levels=levels, precision=prec)
    phi, info = m.solve_pcg(torch.from_numpy(b).cuda(), phi0=torch.from_numpy(phi0).cuda(), tol=0.0, max_iter=4,
                            raise_on_error=False)
    # a residual of b - M phi rounds to about eps 12 n^2 |phi| / |b|; 1e-12 holds at 32^3
    bound = 1e-12 * (n / 32) ** 2
    assert np.max(np.abs(np.array(info.history) - np.array(ref.history)) / ref.history[0]) <= bound
    assert np.linalg.norm(phi.cpu().numpy() - ref.phi) <= bound * np.linalg.norm(ref.phi)


@pytest.mark.parametrize("n,prec", [(64, "mixed"), (128, "mixed"), (256, "fp64"), (256, "mixed"), (512, "fp64"),
                                    (512, "fp32"), (1024, "mixed")])
def test_solution_has_the_reported_residual(n, prec):
    import paper_2607_10983_amd as mg
    torch.manual_seed(n)
    b = torch.randn((n, n, n), device="cuda", dtype=torch.float64) + 0.25
    m = mg.Multigrid(n, levels=n.bit_length() - 2, precision=prec)
    phi, info = m.solve_pcg(b, tol=1e-9, max_iter=30)
    assert 0.0 < info.rel_res <= 1e-9
    b -= b.mean()
    nb = float(b.norm())
    r = phi * -6.0
    for d in range(3):
        for s in (1, -1):
            r += torch.roll(phi, s, d)
    r *= -float(n) ** 2
    r += b
    # two residuals of the same field differ by their rounding only, about
    # eps 12 n^2 |phi| / |b| of the source
    rounding = 2.3e-16 * 12 * n * n * float(phi.norm()) / nb
    assert abs(float(r.norm()) / nb - info.rel_res) <= 2 * rounding + 1e-3 * info.rel_res
    assert abs(float(phi.mean())) <= 1e-12 * float(phi.abs().max())
