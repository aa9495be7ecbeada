"""mg_geometry_bwd_noalloc with a psibar that overlaps an input: refused where
the library's array does not hold the result (blocks would overwrite values
that others still read)."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

MG_OK, MG_ERR_INVALID = 0, 1


def call(n, psi, cbar, sbar, psibar, stream=None):
    from paper_2607_10983_amd import _lib
    p = [ctypes.c_void_p(a) for a in (psi, cbar, sbar, psibar)]
    return _lib.load().mg_geometry_bwd_noalloc(n, 1.0 / n, *p, stream)


@pytest.mark.parametrize("n", [256, 512])
def test_overlap_beyond_the_array_is_refused_on_the_host(n):
    if torch.cuda.is_available():
        pytest.skip("made-up addresses")
    field = 8 * n ** 3
    psi, cbar, sbar = 1 << 40, 1 << 41, 1 << 42
    for psibar in (psi, psi + 8, cbar + 5 * field, cbar - field + 8, sbar, sbar + field - 8):
        assert call(n, psi, cbar, sbar, psibar) == MG_ERR_INVALID


@pytest.mark.gpu
def test_overlap_beyond_the_array_is_refused():
    n = 256
    a = torch.zeros((8, n, n, n), dtype=torch.float64, device="cuda")
    out = torch.full((n, n, n), float("nan"), dtype=torch.float64, device="cuda")
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    psi, cbar, sbar = a[0].data_ptr(), a[1].data_ptr(), a[7].data_ptr()
    for psibar in (psi, a[3].data_ptr(), sbar):
        assert call(n, psi, cbar, sbar, psibar, s) == MG_ERR_INVALID
    assert call(n, psi, cbar, sbar, out.data_ptr(), s) == MG_OK
    torch.cuda.synchronize()
    assert not a.any() and not out.any()  # zero cotangents at the identity map
