"""The fused small levels of a variable-coefficient hierarchy against the CPU
float64 oracle: the visits of the 32^3 level and the single-workgroup tail
of the levels of 16^3 points and fewer.

Inner V-cycle from zero through ``mg_inner_step``: 2e-5 of the largest value
in float (a few dozen float roundings per point and cycle, each 6e-8 of a
value of that size), 1e-12 in double, the bars of every other V-cycle test.
"""
import json
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import mg_oracle as O  # noqa: E402
import workloads as W  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PSI_SCALE = json.load(open(os.path.join(ROOT, "tests", "golden", "psi_scale.json")))["scale"]
BAR = {"mixed": 2e-5, "fp64": 1e-12}


@pytest.fixture(scope="module")
def mgpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_10983_amd as m
    return m


def rounded(a, precision):
    return a if precision == "fp64" else a.astype(np.float32).astype(np.float64)


def check(mgpu, n, levels, smoother, degree, precision):
    psi = PSI_SCALE[str(n)] * W.psi_unit(n)
    C = rounded(O.geometry(psi, 1.0 / n)[0], precision)
    kw = dict(degree=degree) if smoother == "chebyshev" else dict(smoother="jacobi", sweeps=degree)
    mg = mgpu.Multigrid(n, levels=levels, coeff=torch.from_numpy(C).cuda(), precision=precision, **kw)
    H = O.build_hierarchy(n, levels, C=C, **kw)
    r = rounded(np.random.default_rng(n + levels).standard_normal((n, n, n)), precision)
    r = rounded(r - r.mean(), precision)
    ref = O.vcycle(H, 0, np.zeros_like(r), r)
    out = mg.inner_step("vcycle", 0, b=torch.from_numpy(r).cuda()).cpu().numpy()
    err = float(np.max(np.abs(out - ref)) / np.max(np.abs(ref)))
    print(f"{n}^3 {levels} levels {smoother} {degree} {precision}: {err:.2e}", flush=True)
    assert err <= BAR[precision]
    # the cycle inside the solver, whose outer kernel writes the first smoothing step
    phi, info = mg.solve(torch.from_numpy(r).cuda(), tol=0.0, max_cycles=2, raise_on_error=False)
    if precision == "fp64":
        two = O.solve(H, r, tol=0.0, max_cycles=2)
        assert np.max(np.abs(phi.cpu().numpy() - two.phi)) <= 1e-12 * np.max(np.abs(two.phi))


# tails of 16-8-4, 16-8 and 8-4 points a side, alone and below one other level
@pytest.mark.parametrize("n,levels", [(16, 3), (16, 2), (8, 2), (32, 4), (32, 3)])
@pytest.mark.parametrize("smoother,degree", [("chebyshev", 1), ("chebyshev", 2), ("chebyshev", 3), ("chebyshev", 8),
                                             ("jacobi", 2)])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_tail_vcycle(mgpu, n, levels, smoother, degree, precision):
    check(mgpu, n, levels, smoother, degree, precision)


# the visit level alone above the tail, and below one or two row-kernel levels
@pytest.mark.parametrize("n,levels", [(32, 4), (64, 5), (64, 4), (128, 6)])
@pytest.mark.parametrize("smoother,degree", [("chebyshev", 1), ("chebyshev", 2), ("chebyshev", 3), ("chebyshev", 4),
                                             ("chebyshev", 5), ("jacobi", 1), ("jacobi", 3)])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_visit_vcycle(mgpu, n, levels, smoother, degree, precision):
    if n == 128 and degree not in (3, 4):
        pytest.skip("the large grid runs the default degrees only")
    check(mgpu, n, levels, smoother, degree, precision)
