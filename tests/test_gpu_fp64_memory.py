"""Device memory of FP64 plans: that of their atoms, not of every wave the device could hold (42 MB a plan)."""
import pytest

import sputter_inputs as si
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


def test_many_small_plans():
    spx.Plan([si.single_ni(0.5, 1000)], si.Params(), precision=64).run(seed=1)     # loads what every plan shares
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    plans = [spx.Plan([si.single_ni(0.5, 1000)], si.Params(), precision=64) for _ in range(50)]
    used = free - torch.cuda.mem_get_info()[0]
    say(f"50 plans: {used / 2**20:.0f} MiB")
    assert used < 50 * (8 << 20)
    # sizes at which the queue's slots just suffice: a share of the waves rounded up, the smallest of two kernels
    lanes = 256 * torch.cuda.get_device_properties(0).multi_processor_count
    for n in (1, 255, 257, 2047, 2049, 8 * lanes - 1, 8 * lanes, 8 * lanes + 1, 32 * lanes - 1, 32 * lanes, 32 * lanes + 1):
        plan = spx.Plan([si.single_ni(0.4, n)], si.Params(), precision=64)
        C = plan.run(seed=2)["counters"].cpu().numpy()[0]
        assert C[0] == n and C[1] + C[2] + C[3] == n
    del plans
