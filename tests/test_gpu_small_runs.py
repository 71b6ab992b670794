"""Runs small enough that a wave claims less than a full chunk of tickets: sizes around the edges of
the claim's size (8 tickets, a SIMD's share, 128), each particle's record that of the FP64 oracle
(at least 99 % within 1e-3 mm) and the integers bit-identical in every launch shape."""
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


@pytest.mark.parametrize("n", [1, 7, 9, 63, 65, 1023, 8193, 20001])
def test_small_runs_match_the_oracle(n):
    say(f"{n} atoms")
    cfg = [si.single_ni(0.5, n), si.single_ni(2.0, max(1, n // 16))]
    p = si.Params()
    ref = oracle.run(cfg, p, seed=31, records=True)["records"]
    plan = spx.Plan(cfg, p)
    recs = [spx.records_to_numpy(plan.run(seed=31, records=True)["records"])]
    plan.set_launch(5, 64, 2, 4, 4)
    out = plan.run(seed=31, records=True)
    recs.append(spx.records_to_numpy(out["records"]))
    assert np.array_equal(recs[0], recs[1])
    C = out["counters"].cpu().numpy()
    assert np.array_equal(C[:, 0], [n, max(1, n // 16)])
    assert np.array_equal(C[:, 0], C[:, 1] + C[:, 2] + C[:, 3])
    assert np.array_equal(C[:, 1], [int((r["state"] == 1).sum()) for r in np.split(recs[0], [n])])
    m = match_stats(recs[0], ref, 1e-3)
    # a history may miss the tolerance where it passes a decision within rounding: 1 % of them, and one
    assert m["frac"] * m["n"] >= 0.99 * m["n"] - 1, m
