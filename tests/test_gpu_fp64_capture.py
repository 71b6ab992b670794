"""FP64 runs recorded into a caller's graph: a thread per atom, every step tested, nothing shared with the plan's
other runs.  Its outputs are those of the two phases, bit for bit (records, tallies, counters): at
sizes that take both in one kernel at two and three waves per SIMD and a kernel for each, with objects
and arrival tallies, at event caps; and replays that overlap with each other and with eager
runs of the plan do not disturb any of them."""
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


def _chimneys(n, p=0.8):
    k = lambda f: max(1, int(n * f))     # noqa: E731
    return [si.with_chimneys(si.quaternary(p, counts=[k(0.4), k(0.1), k(0.3), k(0.2)]))]


def _scribble(bufs):
    for v in bufs.values():
        if v is not None:
            v.fill_(255 if v.dtype == torch.uint8 else -7)


def _equal(a, b):
    for k, v in a.items():
        if v is not None:
            assert torch.equal(v, b[k]), k


def _captured(plan, runs, **kw):
    """A graph of one run a branch, on streams of their own, with its outputs."""
    bufs = [plan.allocate(**kw) for _ in runs]
    s = [torch.cuda.Stream() for _ in runs]
    s[0].wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s[0]):
        for x in s[1:]:
            x.wait_stream(s[0])
        for x, seed, b in zip(s, runs, bufs):
            plan.run_into(seed, b, stream=x)
        for x in s[1:]:
            s[0].wait_stream(x)
    torch.cuda.synchronize()
    return g, bufs


@pytest.mark.parametrize("name, cfgs, arrivals", [
    ("one atom", [si.single_ni(0.5, 1)], True),
    ("a wave and one", [si.single_ni(2.0, 65), si.single_ni(0.0, 3)], False),
    ("two waves per SIMD", [si.single_ni(0.5, 8 * LANES - 1)], False),
    ("three waves per SIMD", [si.single_ni(0.5, 8 * LANES)], True),
    ("the largest in one kernel", [si.single_ni(0.3, 32 * LANES - 1)], False),
    ("a kernel a phase", [si.single_ni(0.3, 32 * LANES + 11)], True),
    ("unlike pressures", [si.single_ni(0.5, 10 * LANES), si.single_ni(0.1, 6 * LANES + 5)], True),
    ("objects, one kernel", _chimneys(20 * LANES), True),
    ("objects, a kernel a phase", _chimneys(33 * LANES), True),
    ("objects, a kernel a phase, no arrivals", _chimneys(33 * LANES), False)])
def test_equals_the_two_phases(name, cfgs, arrivals):
    say(f"{name}: {sum(c.n_particles for cfg in cfgs for c in cfg.cathodes)} atoms")
    plan = spx.Plan(cfgs, si.Params(), precision=64)
    g, (cap,) = _captured(plan, [19], records=True, arrivals=arrivals)
    _scribble(cap)
    g.replay()
    ref = plan.allocate(records=True, arrivals=arrivals)
    plan.run_into(19, ref)
    torch.cuda.synchronize()
    _equal(ref, cap)


@pytest.mark.parametrize("cap", [1, 2, 129, 130, 261])
def test_event_caps(cap):
    plan = spx.Plan([si.single_ni(2.0, 3000)] + _chimneys(1000, 1.5), si.Params(event_cap=cap), precision=64)
    g, (got,) = _captured(plan, [3], records=True)
    _scribble(got)
    g.replay()
    ref = plan.allocate(records=True)
    plan.run_into(3, ref)
    torch.cuda.synchronize()
    _equal(ref, got)


def test_overlapping_replays():
    say("two branches, an eager run on a third stream and another graph, at the same time")
    plan = spx.Plan([si.single_ni(0.5, 30_000), si.single_ni(1.0, 5_000)], si.Params(), precision=64)
    ref = {}
    for seed in (1, 2, 3, 4):
        ref[seed] = plan.allocate(records=True)
        plan.run_into(seed, ref[seed])
    g, two = _captured(plan, [1, 2], records=True)
    h, (one,) = _captured(plan, [3], records=True)
    eager = plan.allocate(records=True)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(4):
        for x in two + [one, eager]:
            _scribble(x)
        torch.cuda.synchronize()
        g.replay()
        with torch.cuda.stream(a):
            h.replay()
        plan.run_into(4, eager, stream=b)
        torch.cuda.synchronize()
        for seed, x in ((1, two[0]), (2, two[1]), (3, one), (4, eager)):
            _equal(ref[seed], x)
