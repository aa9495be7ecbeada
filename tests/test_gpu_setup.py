"""Setup of a variable-coefficient context on the GPU: geometry, level bounds,
the coarsest dense inverse, and contexts in caller-owned memory.

The row kernels' grids of more than one segment per row (512^3) are checked
through periodicity: a field of period 256 repeated eight times must give the
256^3 result repeated.  Double quantities are compared to 1e-12 of their
largest value (sums of a few dozen terms of that size, well-conditioned 3 x 3
inverses), float ones to one float rounding more, 2e-7.
"""
import ctypes
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


@pytest.fixture(scope="module")
def mgpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_10983_amd as m
    return m


def mesh(n):
    return PSI_SCALE[str(n)] * W.psi_unit(n)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def close(got, ref, tol):
    return float((got - ref).abs().max()) <= tol * float(ref.abs().max())


@pytest.mark.parametrize("n", [8, 64, 128, 256])
def test_geometry(mgpu, n):
    psi = mesh(n)
    Cr, dr = (torch.from_numpy(a) for a in O.geometry(psi, 1.0 / n))
    C, d = mgpu.geometry(dev(psi))
    assert close(C.cpu(), Cr, 1e-12) and close(d.cpu(), dr, 1e-12)
    Cf, df = mgpu.geometry(dev(psi), dtype=torch.float32)
    assert torch.equal(Cf.cpu(), C.float().cpu()) and torch.equal(df, d)


def test_geometry_rows_of_several_segments(mgpu):
    n = 256
    psi = dev(mesh(n))
    C, d = mgpu.geometry(psi)
    C2, d2 = mgpu.geometry(psi.repeat(2, 2, 2), h=1.0 / n)
    for k in range(6):
        assert close(C2[k], C[k].repeat(2, 2, 2), 1e-12)
    assert close(d2, d.repeat(2, 2, 2), 1e-12)


@pytest.mark.parametrize("n,levels", [(16, 2), (16, 3), (64, 5), (128, 5)])
@pytest.mark.parametrize("source", ["coeff32", "coeff64", "psi"])
@pytest.mark.parametrize("precision", ["mixed", "fp64", "fp32"])
def test_level_bounds_and_coarse_inverse(mgpu, n, levels, source, precision):
    psi = mesh(n)
    C = O.geometry(psi, 1.0 / n)[0]
    if source == "coeff32":
        C = C.astype(np.float32)
    kw = {"psi": dev(psi)} if source == "psi" else {"coeff": dev(C)}
    mg = mgpu.Multigrid(n, levels=levels, precision=precision, **kw)
    H = O.build_hierarchy(n, levels, psi=psi) if source == "psi" else \
        O.build_hierarchy(n, levels, C=C.astype(np.float64))
    ref = [lev.cheb.lmax for lev in H.levels][:-1]
    assert np.allclose(mg.level_lmax()[:-1], ref, rtol=1e-12, atol=0)
    nc = n >> (levels - 1)
    r = np.random.default_rng(3).standard_normal((nc, nc, nc))
    e = O.coarse_solve(H.levels[-1], r)
    assert np.max(np.abs(mg.coarse_solve(dev(r)).cpu().numpy() - e)) <= 1e-12 * np.max(np.abs(e))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_bounds_of_several_segments(mgpu, dtype):
    n = 256
    C = mgpu.geometry(dev(mesh(n)), dtype=dtype)[0]
    prec = "mixed" if dtype == torch.float32 else "fp64"
    one = mgpu.Multigrid(n, levels=6, coeff=C, precision=prec, h=1.0 / n)
    two = mgpu.Multigrid(2 * n, levels=7, coeff=C.repeat(1, 2, 2, 2), precision=prec, h=1.0 / n)
    # a period of the fine field is a period of every restricted one
    assert np.allclose(two.level_lmax()[:5], one.level_lmax()[:5], rtol=1e-12, atol=0)


@pytest.mark.parametrize("source", ["flat", "coeff", "psi"])
def test_library_and_caller_memory_give_the_same_solution(mgpu, source):
    L = mgpu._lib
    lib = L.load()
    n = 32
    psi = dev(mesh(n))
    C = mgpu.geometry(psi)[0]
    b = dev(W.flat_source(n, 5))
    kw = {"coeff": {"coeff": C}, "psi": {"psi": psi}}.get(source, {})
    phi, info = mgpu.Multigrid(n, **kw).solve(b, tol=1e-9)
    p = L.MgParams()
    lib.mg_params_default(ctypes.byref(p), n)
    h = ctypes.c_void_p()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    if source == "psi":
        st = lib.mg_create_psi(ctypes.byref(p), ctypes.c_void_p(psi.data_ptr()), stream, ctypes.byref(h))
    else:
        st = lib.mg_create(ctypes.byref(p), ctypes.c_void_p(C.data_ptr()) if source == "coeff" else None,
                           L.MG_DTYPE_F64, stream, ctypes.byref(h))
    assert st == L.MG_OK
    own = torch.zeros_like(b)
    st = lib.mg_solve(h, ctypes.c_void_p(own.data_ptr()), ctypes.c_void_p(b.data_ptr()), 1e-9, 50, None)
    assert st == L.MG_OK
    assert lib.mg_destroy(h) == L.MG_OK
    assert torch.equal(own, phi)


def test_caller_memory_is_checked(mgpu):
    L = mgpu._lib
    lib = L.load()
    p = L.MgParams()
    lib.mg_params_default(ctypes.byref(p), 16)
    keep, setup = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.mg_workspace_bytes(ctypes.byref(p), 4, ctypes.byref(keep), ctypes.byref(setup)) == L.MG_ERR_INVALID
    assert lib.mg_workspace_bytes(ctypes.byref(p), L.MG_SOURCE_PSI, ctypes.byref(keep), ctypes.byref(setup)) == L.MG_OK
    mem = torch.empty(keep.value, dtype=torch.uint8, device="cuda")
    tmp = torch.empty(setup.value, dtype=torch.uint8, device="cuda")
    psi = dev(mesh(16))
    h = ctypes.c_void_p()
    args = lambda k, t: (ctypes.byref(p), L.MG_SOURCE_PSI, ctypes.c_void_p(psi.data_ptr()),  # noqa: E731
                         ctypes.c_void_p(mem.data_ptr()), ctypes.c_size_t(k), ctypes.c_void_p(tmp.data_ptr()),
                         ctypes.c_size_t(t), None, ctypes.byref(h))
    assert lib.mg_create_in(*args(keep.value - 1, setup.value)) == L.MG_ERR_INVALID
    assert lib.mg_create_in(*args(keep.value, setup.value - 1)) == L.MG_ERR_INVALID
    assert lib.mg_create_in(*args(keep.value, setup.value)) == L.MG_OK
    assert lib.mg_destroy(h) == L.MG_OK
