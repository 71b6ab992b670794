"""A run of a plan of many segments: the host's part does not grow with them (it took 125 us more for 80000
segments when it went over all of them; three times that of one chamber is allowed)."""
import time

import pytest

import sputter_inputs as si
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


def _enqueue_us(chambers):
    plan = spx.Plan([si.quaternary(0.5, counts=[5] * 4, grid_n=4) for _ in range(chambers)], si.Params())
    bufs = plan.allocate()
    best = 1e9
    for _ in range(40):
        t = time.perf_counter()
        plan.run_into(3, bufs)
        best = min(best, time.perf_counter() - t)
        torch.cuda.synchronize()
    return 1e6 * best


def test_enqueue_time():
    one, many = _enqueue_us(1), _enqueue_us(20000)
    say(f"4 segments {one:.0f} us, 80000 {many:.0f} us")
    assert many < 3 * one
