"""What the autotuner may change for a plan whose runs take both phases in one kernel, and for one whose
runs take a kernel for each."""
import pytest

import sputter_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("cfgs", [
    [si.single_ni(0.5, 300_000)], [si.with_chimneys(si.quaternary(0.5, counts=[30_000, 10_000, 20_000, 15_000]))]])
def test_autotune_times_the_kernel_that_runs(cfgs):
    # blocks and threads are those of the two kernels that such a plan does not launch: they stay
    plan = spx.Plan(cfgs, si.Params())
    plan.set_launch(0, 128, 4, 16, 8)
    before = plan.launch
    ref = plan.run(seed=4, records=True)
    times = plan.phase_times()
    after = plan.autotune()
    assert plan.phase_times() == times
    assert (after["blocks"], after["threads"]) == (before["blocks"], before["threads"])
    out = plan.run(seed=4, records=True)
    for k in ("counts", "counters", "records"):
        assert torch.equal(out[k], ref[k]), k


def test_autotune_of_a_long_run_picks_a_shape():
    plan = spx.Plan([si.single_ni(0.1, 6_000_000)], si.Params())
    ref = plan.run(seed=4)
    launch = plan.autotune()
    assert launch["threads"] in (256, 512, 1024)
    assert torch.equal(plan.run(seed=4)["counts"], ref["counts"])
