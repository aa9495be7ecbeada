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
