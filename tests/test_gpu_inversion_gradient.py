"""A measured library that takes part in a gradient: the inversion's outputs are values without one."""
import pytest

import sputter_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


def test_measured_library_in_a_gradient():
    x = [11.0, 12.0, 13.0]
    plan = spx.Plan([si.ternary(0.5, t, n_particles=1000, grid_n=40) for t in x], si.Params())
    g = torch.Generator(device="cuda").manual_seed(1)
    prof = torch.rand(plan.n_bins, dtype=torch.float64, device="cuda", generator=g) + 0.5
    comp = si.ternary_composition_inputs()
    meas = torch.rand(50, 3, device="cuda", generator=g)
    cen = spx.area_centres(50)
    ref = spx.invert_sweep(plan, {"profiles": prof}, x, comp, meas, centres=cen)
    got = spx.invert_sweep(plan, {"profiles": prof}, x, comp, meas.clone().requires_grad_(True), centres=cen)
    for k, v in ref.items():
        assert not got[k].requires_grad, k
        assert torch.equal(got[k], v) or (torch.isnan(got[k]).all() and torch.isnan(v).all()), k
