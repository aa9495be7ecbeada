"""mg_destroy gives the caller's memory back only when the work of the context is
done, on the streams it had before its last one too."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("switch", [False, True])
def test_destroy_waits_for_earlier_streams(switch):
    from paper_2607_10983_amd import _lib as L
    lib = L.load()
    n = 256
    p = L.MgParams()
    lib.mg_params_default(ctypes.byref(p), n)
    p.precision = L.MG_FP64
    size, setup = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.mg_workspace_bytes(ctypes.byref(p), L.MG_SOURCE_FLAT, ctypes.byref(size), ctypes.byref(setup)) == L.MG_OK
    keep = torch.empty(size.value, dtype=torch.uint8, device="cuda")
    b = torch.randn((n, n, n), dtype=torch.float64, device="cuda")
    phi = torch.zeros_like(b)
    torch.cuda.synchronize()
    a, other = torch.cuda.Stream(), torch.cuda.Stream()
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    h = ctypes.c_void_p()
    assert lib.mg_create_in(ctypes.byref(p), L.MG_SOURCE_FLAT, None, ptr(keep), size, None, ctypes.c_size_t(0),
                            ctypes.c_void_p(a.cuda_stream), ctypes.byref(h)) == L.MG_OK
    for _ in range(60):  # about 40 ms of work, enqueued in a few
        assert lib.mg_vcycle(h, ptr(phi), ptr(b), None) == L.MG_OK
    if switch:
        assert lib.mg_set_stream(h, ctypes.c_void_p(other.cuda_stream)) == L.MG_OK
    assert lib.mg_destroy(h) == L.MG_OK
    assert a.query()
