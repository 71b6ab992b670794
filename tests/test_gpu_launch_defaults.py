"""Launch parameters that set_launch restores without arguments: those of a plan that is not tuned."""
import pytest

import sputter_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


def test_set_launch_without_arguments_restores_the_untuned_plan():
    plan = spx.Plan([si.single_ni(0.5, 1000)], si.Params())
    fresh = plan.launch
    plan.set_launch(0, 512, 2, 12, 16)
    assert plan.set_launch() == fresh
