"""Squares beyond the grid, at any distance and in any direction, infinitely far among them: no bin, value 0,
in the time of any other call; the squares beside them are as they are without (1e-13 relative)."""
import numpy as np
import pytest

import oracle
import sputter_inputs as si
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("nu, nv, hw", [(50, 50, 0.4), (50, 50, 2.25), (200, 200, 2.25), (49, 124, 91.2), (1, 300, 20.0), (300, 1, 20.0)])
@pytest.mark.parametrize("far", [150.0, 1e6, 2147483647.0, 1e12, 1e300, np.inf])
def test_far_squares(nu, nv, hw, far):
    say(f"{nu} x {nv} bins, half width {hw}, squares {far} mm away")
    g = si.Grid(nu=nu, nv=nv, half_u=50.0, half_v=45.0)
    prof = np.random.default_rng(nu).uniform(0.5, 1.5, (2, nv, nu))
    near = np.array([[0.0, 0.0], [12.34, -5.67], [49.0, 44.0]])
    out = np.array([[far, 0.0], [-far, 0.0], [0.0, far], [0.0, -far], [far, far], [-far, far], [far, -far], [-far, -far]])
    cen = np.concatenate([near, out, near])
    got = spx.area_gather(torch.as_tensor(prof, device="cuda"), g, cen, hw).cpu().numpy()
    ref = np.stack([oracle.area_gather(p, g, near, hw) for p in prof])
    assert np.allclose(got[:, :3], ref, rtol=1e-13, atol=0) and np.allclose(got[:, -3:], ref, rtol=1e-13, atol=0)
    assert (got[:, 3:-3] == 0).all()
