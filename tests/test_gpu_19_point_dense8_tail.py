"""Which 19-point hierarchies with an 8^3 coarsest level run their 16^3 level in
the single-workgroup tail: with fewer smoothing steps the launches are faster,
and a cycle has to be bit for bit that of MG_OPT_NO_TAIL.  The tail itself
multiplies by 1 / D where the launches divide, so its cycles differ in the last
bits.  Both sides of every threshold (it depends on the type and on how many
levels lie above)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

MG_OPT_NO_TAIL = 4


@pytest.mark.parametrize("precision,n,degree,tail", [
    ("mixed", 16, 3, False), ("mixed", 16, 4, True), ("mixed", 32, 3, False), ("mixed", 32, 4, True),
    ("mixed", 64, 8, False), ("fp32", 64, 4, False),
    ("fp64", 16, 4, False), ("fp64", 16, 5, True), ("fp64", 64, 4, False), ("fp64", 64, 5, True),
    ("fp64", 128, 6, False), ("fp64", 128, 7, True),
    ("mixed", 64, -11, False), ("mixed", 64, -12, True),  # Jacobi sweeps
])
def test_route_of_an_8_cubed_coarsest_level(precision, n, degree, tail):
    import paper_2607_10983_amd as mg
    g = torch.Generator(device="cuda").manual_seed(n)
    psi = 0.02 * torch.randn((n, n, n), generator=g, device="cuda", dtype=torch.float64) / n ** 2
    b = torch.randn((n, n, n), generator=g, device="cuda", dtype=torch.float64)
    kw = dict(degree=degree) if degree > 0 else dict(smoother="jacobi", sweeps=-degree)
    cycles = [mg.Multigrid(n, levels=n.bit_length() - 3, psi=psi, precision=precision, options=o, **kw)
              .inner_step("vcycle", 0, b=b) for o in (0, MG_OPT_NO_TAIL)]
    assert torch.equal(*cycles) == (not tail)
