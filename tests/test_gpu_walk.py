"""The diffusive walk in groups of steps: event caps at the edges of a group's reach (129 events),
where waves switch between groups and single steps, and deferral thresholds from one held step to
the whole wave.  The bar is the transport's: integers bit-identical across launch shapes, states and
end points those of the FP64 oracle (at least 99.5 % and 99 % within 1e-3 mm)."""
import numpy as np
import pytest

import oracle
import sputter_inputs as si
from parity import match_stats, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("cap", [1, 2, 40, 128, 129, 130, 131, 260])
def test_caps_at_the_edges_of_a_group(cap):
    say(f"event cap {cap}")
    p = si.Params(event_cap=cap)
    cfg = [si.single_ni(2.0, 1500), si.with_chimneys(si.quaternary(1.0, counts=[300, 200, 100, 150]))]
    ref = oracle.run(cfg, p, seed=23, records=True)["records"]
    plan = spx.Plan(cfg, p)
    recs = []
    for blocks, threads, refill, defer in ((0, 256, 8, 8), (2, 64, 1, 1), (3, 1024, 16, 64)):
        plan.set_launch(blocks, threads, refill, 16, defer)
        recs.append(spx.records_to_numpy(plan.run(seed=23, records=True)["records"]))
    for r in recs[1:]:
        assert np.array_equal(r, recs[0])
    rec = recs[0]
    capped = rec["state"] == 3
    assert rec["events"].max() == cap and np.all(rec["events"][capped] == cap)
    m = match_stats(rec, ref, 1e-3)
    assert m["same_state"] >= 0.995 and m["frac"] >= 0.99, m
    same = rec["state"] == ref[:, 3].astype(np.uint32)
    assert np.mean(rec["diffusive"][same] == ref[same, 6].astype(np.uint32)) >= 0.99
