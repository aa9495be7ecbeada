"""Force readout on rows of several segments (512^3): a potential of period
256 repeated eight times must give the 256^3 force repeated.  Both grids
evaluate the same sums of the same values; the bound allows two roundings of
the largest one (double: 2^-51, float: 2^-22)."""
import json
import os

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import workloads as W  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PSI_SCALE = json.load(open(os.path.join(ROOT, "tests", "golden", "psi_scale.json")))["scale"]


@pytest.mark.parametrize("curv", [False, True])
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 2.0 ** -22), (torch.float64, 2.0 ** -51)])
def test_force_is_periodic(curv, dtype, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_10983_amd as mgpu
    n, h = 256, 1.0 / 256
    phi = torch.from_numpy(W.flat_source(n, 1)).cuda()
    psi = torch.from_numpy(PSI_SCALE[str(n)] * W.psi_unit(n)).cuda() if curv else None
    one = mgpu.accel(phi, psi, scale=0.45, h=h, dtype=dtype)
    two = mgpu.accel(phi.repeat(2, 2, 2), psi.repeat(2, 2, 2) if curv else None, scale=0.45, h=h, dtype=dtype)
    for k in range(3):
        assert float((two[k] - one[k].repeat(2, 2, 2)).abs().max()) <= tol * float(one[k].abs().max())
