"""Phase times are those of the plan's last run of its own, whatever replays of it a caller's graph makes."""
import pytest

import sputter_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("n", [20_000, 6_000_000])
def test_phase_times_outlast_captured_replays(n):
    plan = spx.Plan([si.single_ni(0.5, n)], si.Params())
    bufs = plan.allocate()
    plan.run_into(1, bufs)
    times = plan.phase_times()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        plan.run_into(2, bufs, stream=s)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert plan.phase_times() == times
