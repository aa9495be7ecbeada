"""Reverse mode of the geometry in chunks of 16 planes, which every grid of 128^3
points and more runs (smaller ones: chunks of 4), against references that do not
go through the same traversal.

The oracle comparison allows 1e-12 of the largest value, the bar of the oracle
tests at 16^3: a sum of 19 terms of that size, each a few dozen roundings from a
well-conditioned 3 x 3 inverse.  The others are exact: a point's operations do
not depend on the chunk or the tile it falls in.
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


def inputs(n, seed):
    rng = np.random.default_rng(seed)
    return PSI_SCALE[str(n)] * W.psi_unit(n), rng.standard_normal((6, n, n, n)), rng.standard_normal((n, n, n))


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def test_against_the_oracle_at_128():
    import paper_2607_10983_amd as mg
    n = 128
    psi, cbar, sbar = inputs(n, 1)
    got = mg.geometry_bwd(dev(psi), dev(cbar), dev(sbar)).cpu().numpy()
    want = O.geometry_bwd(psi, cbar, sbar, 1.0 / n)
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()


# 64^3 runs chunks of 4 planes, 128^3 and 256^3 of 16
@pytest.mark.parametrize("n", [64, 128])
@pytest.mark.parametrize("with_sbar", [True, False])
def test_a_repeated_field_gives_the_repeated_result(n, with_sbar):
    import paper_2607_10983_amd as mg
    psi, cbar, sbar = (dev(a) for a in inputs(n, 2))
    one = mg.geometry_bwd(psi, cbar, sbar if with_sbar else None, h=1.0 / n)
    two = mg.geometry_bwd(psi.repeat(2, 2, 2), cbar.repeat(1, 2, 2, 2),
                          sbar.repeat(2, 2, 2) if with_sbar else None, h=1.0 / n)
    assert torch.equal(two, one.repeat(2, 2, 2))


@pytest.mark.parametrize("entry", ["mg_geometry_bwd", "mg_geometry_bwd_noalloc"])
def test_result_may_replace_an_input_at_128(entry):
    import paper_2607_10983_amd as mg
    from paper_2607_10983_amd import _lib
    n = 128
    given = [dev(a) for a in inputs(n, 3)]
    want = mg.geometry_bwd(*given)
    for which in range(3):
        a = [t.clone() for t in given]
        out = a[which][5] if which == 1 else a[which]
        p = [ctypes.c_void_p(t.data_ptr()) for t in a]
        st = getattr(_lib.load(), entry)(n, 1.0 / n, *p, ctypes.c_void_p(out.data_ptr()),
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == _lib.MG_OK
        torch.cuda.synchronize()
        assert torch.equal(out, want)
