"""The FP64 path's two phases at sizes around their edges (one atom, a claim, a full wave), event caps at
the edges of a group of steps, absorbing objects, and a plan of two rounds: each record the oracle's
(at least 99.9 % within 1e-6 mm, the bar of the FP64 path), the tallies those of the records."""
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


def _check(cfg, p, seed):
    ref = oracle.run(cfg, p, seed=seed, records=True)
    out = spx.Plan(cfg, p, precision=64).run(seed=seed, records=True, arrivals=True)
    rec, C = spx.records_to_numpy(out["records"]), out["counters"].cpu().numpy()
    # a history may leave the oracle's where it passes a decision within rounding: 0.1 % of them, and one
    m = match_stats(rec, ref["records"], 1e-6)
    assert m["frac"] * m["n"] >= 0.999 * m["n"] - 1, m
    assert np.array_equal(C[:, 0], C[:, 1] + C[:, 2] + C[:, 3])
    assert C[:, 1].sum() == (rec["state"] == 1).sum() and C[:, 5].sum() == rec["diffusive"].sum()
    # every diffusive step counts as tested: those that ended in the gas and the last one of a walk that ended
    thermal = (ref["records"][:, 6] > 0) & (rec["state"] != 3)
    assert abs(int(C[:, 7].sum()) - int(rec["diffusive"].sum()) - int(thermal.sum())) <= 0.01 * len(rec) + 1
    assert out["arrival_energy"].sum().item() == C[:, 1].sum() == out["counts"].sum().item()
    return rec


@pytest.mark.parametrize("n", [1, 8, 65, 4000])
def test_sizes(n):
    say(f"FP64, {n} atoms")
    _check([si.single_ni(0.5, n), si.single_ni(2.0, max(1, n // 8))], si.Params(), 41)


@pytest.mark.parametrize("cap", [1, 129, 130, 260])
def test_caps(cap):
    say(f"FP64, event cap {cap}")
    rec = _check([si.single_ni(2.0, 800), si.with_chimneys(si.quaternary(1.0, counts=[200, 60, 70, 80]))],
                 si.Params(event_cap=cap), 43)
    assert rec["events"].max() == cap and np.all(rec["events"][rec["state"] == 3] == cap)


def test_two_rounds():
    n = (1 << 24) + 1001
    say(f"FP64, {n} atoms at 0 Pa in two rounds")
    out = spx.Plan([si.single_ni(0.0, n)], si.Params(), precision=64).run(seed=5, records=True)
    C = out["counters"].cpu().numpy()[0]
    assert C[0] == n and C[1] + C[2] == n
    words = out["records"].view(torch.int32).view(n, 14)
    bins = words[:, 9][words[:, 8] == 1].to(torch.int64)
    assert torch.equal(torch.bincount(bins, minlength=2500), out["counts"])
