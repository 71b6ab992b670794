"""Instances of the transport kernels that other sizes and options do not reach: passes of a wave over its
own slots of the scratch array with objects and arrival tallies, several rounds of a kernel per phase
with atoms in the queue of each, in FP32 and FP64.  A history does not depend on its lane: outputs
equal to the bit."""
import pytest

import sputter_inputs as si
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402

# one ticket per lane of one wave per SIMD
LANES = 256 * torch.cuda.get_device_properties(0).multi_processor_count


def _system(objects, n):
    counts = [int(0.4 * n), int(0.1 * n), int(0.3 * n), n - int(0.4 * n) - int(0.1 * n) - int(0.3 * n)]
    cfg = si.quaternary(0.5, counts=counts)
    return [si.with_chimneys(cfg) if objects else cfg]


def _scribble(bufs):
    for v in bufs.values():
        if v is not None:
            v.fill_(255 if v.dtype == torch.uint8 else -7)


def _equal(a, b):
    for k, v in a.items():
        if v is not None:
            assert torch.equal(v, b[k]), k


@pytest.mark.parametrize("arrivals", [False, True])
@pytest.mark.parametrize("objects", [False, True])
@pytest.mark.parametrize("small_grid", [False, True])
def test_scratch_array(objects, arrivals, small_grid):
    # 1 398 080 slots: in one kernel the waves use theirs several times over, in two there are three rounds
    say(f"3e6 atoms, objects {objects}, arrivals {arrivals}, {'a kernel a phase' if small_grid else 'one kernel'}")
    plan = spx.Plan(_system(objects, 3_000_000), si.Params())
    ref, got = (plan.allocate(records=True, arrivals=arrivals) for _ in range(2))
    plan.run_into(11, ref)
    if small_grid:
        plan.set_launch(LANES // 512, 256, 4, 16, 8)
    for _ in range(2):
        _scribble(got)
        plan.run_noalloc_into(11, got)
        torch.cuda.synchronize()
        _equal(ref, got)


def test_two_rounds_in_fp64():
    n = (1 << 24) + 1001
    say(f"FP64, {n} atoms at 0.3 Pa in two rounds, and with a thread an atom")
    plan = spx.Plan([si.single_ni(0.3, n)], si.Params(), precision=64)
    ref, got = plan.allocate(arrivals=True), plan.allocate(arrivals=True)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        plan.run_into(8, got, stream=s)
    _scribble(got)
    g.replay()
    plan.run_into(8, ref)
    torch.cuda.synchronize()
    _equal(ref, got)
    assert ref["counters"].view(-1)[0].item() == n and ref["counters"].view(-1)[6].item() > n // 5
