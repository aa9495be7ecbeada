"""The binding around a context, with the library or the device stood in for:
calls on a closed context and a library allocation that finds no memory."""
import ctypes
import types

import pytest

torch = pytest.importorskip("torch")

import paper_2607_10983_amd as mg  # noqa: E402
from paper_2607_10983_amd import _lib as L  # noqa: E402


def context(monkeypatch, handle=None):
    """A Multigrid object without a device, created on a stream other than the current one."""
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=0))
    m = mg.Multigrid.__new__(mg.Multigrid)
    m.n, m.levels, m._ctx, m._keep, m._stream = 8, 2, handle, None, object()
    return m


def test_a_closed_context_on_another_stream_reports_an_invalid_call(monkeypatch):
    m = context(monkeypatch)
    x = torch.zeros((8, 8, 8), dtype=torch.float64)
    with pytest.raises(mg.MGError) as e:
        m._run("mg_solve", x, x.clone(), 1e-6, 3, True, True)
    assert e.value.status == L.MG_ERR_INVALID


class Library:
    """Reports MG_ERR_NOMEM for the first call of every entry point and MG_OK for the next."""

    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        if not name.startswith("mg_"):
            raise AttributeError(name)
        if name == "mg_last_error":
            return lambda ctx: b""

        def entry(*args):
            if name == "mg_set_stream":
                return L.MG_OK
            self.calls.append(name)
            return L.MG_ERR_NOMEM if self.calls.count(name) == 1 else L.MG_OK
        return entry


@pytest.mark.parametrize("call", [
    lambda m, x: m._run("mg_solve_pcg", x, x, 1e-6, 3, True, True),
    lambda m, x: m.smooth(x, x),
    lambda m, x: m.residual_restrict(x, x),
])
def test_memory_the_allocator_holds_is_given_back_before_an_allocation_fails(monkeypatch, call):
    m = context(monkeypatch, handle=ctypes.c_void_p(1))
    lib, emptied = Library(), []
    monkeypatch.setattr(L, "load", lambda: lib)
    monkeypatch.setattr(torch.cuda, "empty_cache", lambda: emptied.append(list(lib.calls)))
    monkeypatch.setattr(mg, "_check_field", lambda *a, **k: None)
    call(m, torch.zeros((8, 8, 8), dtype=torch.float64))
    assert len(lib.calls) == 2 and emptied == [lib.calls[:1]]
    m._ctx = None
