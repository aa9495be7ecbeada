"""The coarsest dense solve of coefficients whose operator is indefinite: finite
cells with positive diagonal components, as a context accepts them, but large
off-diagonals.  One leading minor of the matrix is brought next to zero by
scaling the off-diagonals, so an elimination in the natural order without
pivoting meets a vanishing pivot although the matrix is well conditioned."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import mg_oracle as O  # noqa: E402


def shifted(C, n):
    """The matrix whose inverse the coarsest solve projects: M - s 1 1^T / N."""
    M = O.dense_from_apply(lambda u: O.apply_var(u, C, 1.0 / n), n)
    return M - np.abs(np.diag(M)).mean() / n ** 3


def near_singular_minor(n, seed):
    """C with a leading minor next to zero, and its matrix."""
    rng = np.random.default_rng(seed)
    diag, off = rng.uniform(0.5, 1.5, (3, n, n, n)), rng.standard_normal((3, n, n, n))
    # linear in the scale of the off-diagonals
    A0 = shifted(np.concatenate([diag, 0 * off]), n)
    A1 = shifted(np.concatenate([diag, off]), n) - A0
    sign = lambda a, k: np.linalg.slogdet((A0 + a * A1)[:k, :k])[0]  # noqa: E731
    lo, hi = 2.0, 2.5
    k = next(k for k in range(n ** 3 // 4, n ** 3) if sign(lo, k) != sign(hi, k))
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if sign(mid, k) == sign(lo, k) else (lo, mid)
    return np.concatenate([diag, lo * off]), A0 + lo * A1


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_coarse_solve_of_an_indefinite_operator(precision):
    import paper_2607_10983_amd as mg
    n = 8
    C, A = near_singular_minor(n, 4)
    w = np.linalg.eigvalsh(A)
    cond = np.abs(w).max() / np.abs(w).min()
    assert w.min() < 0 < w.max() and cond < 1e5
    r = np.random.default_rng(5).standard_normal((n, n, n))
    r -= r.mean()
    e = np.linalg.solve(A, r.ravel())
    e -= e.mean()
    ctx = mg.Multigrid(n, levels=1, coeff=torch.from_numpy(C).cuda(), precision=precision)
    got = ctx.coarse_solve(torch.from_numpy(r).cuda()).cpu().numpy().ravel()
    # a pivoted elimination: rounding times the condition, a growth of up to 64 allowed for
    assert np.abs(got - e).max() <= 64 * np.finfo(float).eps * cond * np.abs(e).max()
