"""Which 19-point hierarchies with an 8^3 coarsest level run their 16^3 level in
the single-workgroup tail: below eight steps a pass the launches are faster, and
a cycle has to be bit for bit that of MG_OPT_NO_TAIL.  The tail itself multiplies
by 1 / D where the launches divide, so its cycles differ in the last bits."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

MG_OPT_NO_TAIL = 4


@pytest.mark.parametrize("n,levels", [(16, 2), (32, 3)])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("kw,tail", [(dict(degree=1), False), (dict(degree=3), False), (dict(degree=7), False),
                                     (dict(degree=8), True), (dict(smoother="jacobi", sweeps=7), False),
                                     (dict(smoother="jacobi", sweeps=8), True)])
def test_route_of_an_8_cubed_coarsest_level(n, levels, precision, kw, tail):
    import paper_2607_10983_amd as mg
    g = torch.Generator(device="cuda").manual_seed(n)
    psi = 0.02 * torch.randn((n, n, n), generator=g, device="cuda", dtype=torch.float64) / n ** 2
    b = torch.randn((n, n, n), generator=g, device="cuda", dtype=torch.float64)
    cycles = [mg.Multigrid(n, levels=levels, psi=psi, precision=precision, options=o, **kw).inner_step("vcycle", 0, b=b)
              for o in (0, MG_OPT_NO_TAIL)]
    assert torch.equal(*cycles) == (not tail)
