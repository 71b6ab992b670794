"""Runs that take both phases in one kernel: sizes at the edges of its waves per SIMD, of its blocks and of
its range, against the same run as a kernel per phase (which a grid of less than a wave per SIMD
selects).  A history does not depend on the lane that takes it: every output is equal to the bit."""
from dataclasses import replace

import numpy as np
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
KEYS = ("counts", "counters", "records", "profiles", "arrival_energy", "arrival_angle", "energy_sum")


def _systems(n):
    k = lambda f: max(1, int(n * f))     # noqa: E731
    return {
        "single": [si.single_ni(0.5, n)],
        "dense": [si.single_ni(2.0, n)],
        "pressures": [si.single_ni(0.5, n - 2 * (n // 3)), si.single_ni(0.0, n // 3), si.single_ni(2.0, n // 3)],
        "chimneys": [si.with_chimneys(si.quaternary(0.8, counts=[k(0.4), k(0.1), k(0.3), k(0.2)]))],
    }


@pytest.mark.parametrize("arrivals", [False, True])
@pytest.mark.parametrize("system, n", [
    ("single", 1), ("single", 255), ("single", 4097), ("single", 4 * LANES - 1), ("single", 4 * LANES),
    ("single", 20 * LANES), ("dense", 3 * LANES + 17), ("pressures", 3), ("pressures", 16 * LANES - 1),
    ("pressures", 16 * LANES), ("chimneys", 1000), ("chimneys", 5 * LANES)])
def test_equals_two_kernels(system, n, arrivals):
    say(f"{system}, {n} atoms, arrivals {arrivals}")
    plan = spx.Plan(_systems(n)[system], si.Params())
    outs = [plan.run(seed=77, records=True, arrivals=arrivals)]
    tb, td = plan.phase_times()
    assert tb > 0 and td > 0
    if n == 255:
        plan.autotune()
        assert plan.phase_times() == (tb, td)
    plan.set_launch(LANES // 512, 256, 4, 16, 8)
    outs.append(plan.run(seed=77, records=True, arrivals=arrivals))
    torch.cuda.synchronize()
    for key in KEYS:
        if key in outs[0] and outs[0][key] is not None:
            assert torch.equal(outs[0][key], outs[1][key]), key
    C = outs[0]["counters"]
    assert C[:, 0].sum().item() == sum(c.n_particles for cfg in _systems(n)[system] for c in cfg.cathodes)


@pytest.mark.parametrize("n", [7, 5000, 100001])
def test_fp64_equals_two_kernels(n):
    # a particle's history depends on its number, not on how many there are
    say(f"FP64, {n} atoms")
    big = 17 * LANES
    recs = []
    for k in (n, big):
        cfg = [si.single_ni(0.5, k), si.single_ni(0.1, 10)]
        recs.append(spx.records_to_numpy(spx.Plan(cfg, si.Params(), precision=64).run(seed=5, records=True)["records"]))
    assert np.array_equal(recs[0][:n], recs[1][:n])


@pytest.mark.parametrize("n", [1398080, 1398081, 3000000, 80 * LANES + 5])
def test_scratch_array(n):
    # its 1 398 080 slots: all of them, then passes of a wave over its own slots, then two rounds of those
    say(f"{n} atoms from the scratch array")
    plan = spx.Plan([si.single_ni(0.5, n)], si.Params())
    ref = plan.run(seed=9, records=True)
    got = plan.allocate(records=True)
    plan.run_noalloc_into(9, got)
    torch.cuda.synchronize()
    for key in ("counts", "counters", "records", "profiles"):
        assert torch.equal(got[key].view(-1), ref[key].view(-1)), key


@pytest.mark.parametrize("arrivals", [False, True])
def test_the_largest_tally_and_counters_in_lds(arrivals):
    # 256 segments (their counters 16 384 bytes) of 48 bins (the tally 49 152 bytes): all that a block may keep
    say("256 segments of 48 bins")
    cfgs = []
    for c in range(64):
        cfg = si.quaternary(0.5 + 0.005 * c, counts=[40, 20, 30, 10])
        cfgs.append(replace(cfg, grid=replace(cfg.grid, nu=8, nv=6)))
    plan = spx.Plan(cfgs, si.Params())
    assert plan.n_segments == 256 and plan.n_bins == 12288
    outs = [plan.run(seed=3, arrivals=arrivals)]
    plan.set_launch(LANES // 512, 256, 4, 16, 8)
    outs.append(plan.run(seed=3, arrivals=arrivals))
    for key in KEYS:
        if outs[0].get(key) is not None:
            assert torch.equal(outs[0][key], outs[1][key]), key
    assert outs[0]["counters"].sum(0)[0].item() == 6400


def test_fp64_segments_meet_in_a_wave():
    # shares of many tickets, each segment's boundary inside one: the records of segments run alone
    say("FP64, boundaries of segments inside the waves' shares")
    counts = [150001, 7, 60013, 120002]
    cfg = si.quaternary(0.5, counts=counts)
    both = spx.records_to_numpy(spx.Plan([cfg], si.Params(), precision=64).run(seed=6, records=True)["records"])
    more = si.quaternary(0.5, counts=[4 * c for c in counts])
    far = spx.records_to_numpy(spx.Plan([more, si.single_ni(0.1, 14 * LANES)], si.Params(),
                                        precision=64).run(seed=6, records=True)["records"])
    first, first4 = 0, 0
    for c in counts:
        assert np.array_equal(both[first:first + c], far[first4:first4 + c])
        first, first4 = first + c, first4 + 4 * c
