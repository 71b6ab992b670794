"""Absorbing objects in the walk of a drained wave's last walkers, where the lanes of a walker's span share
them: numbers of objects around the span widths (none next to many, 1 .. 32), both precisions.  The
records are the oracle's (FP32 at least 99 % within 1e-3 mm, FP64 99.9 % within 1e-6 mm) and do not
depend on the launch shape."""
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


def _ring(n):
    """n small discs, rectangles and tubes on a ring between target and substrate, clear of the axis."""
    out = []
    for k in range(n):
        a = 2 * np.pi * k / n
        c = (60.0 * np.cos(a), 60.0 * np.sin(a), 130.0 + 2.0 * (k % 5))
        kind = ("disc", "rect", "tube")[k % 3]
        out.append(si.Absorber(kind, center=c, normal=(0.0, 0.0, 1.0), half_u=4.0, half_v=3.0, length=12.0))
    return out


@pytest.mark.parametrize("n", [1, 2, 3, 5, 17, 32])
def test_objects_shared_by_a_span(n):
    say(f"{n} objects")
    cfgs = [si.single_ni(0.5, 1500), si.single_ni(1.5, 600)]
    cfgs[0].absorbers = _ring(n)
    cfgs.append(si.single_ni(1.0, 300))          # no objects, in the same waves
    p = si.Params()
    ref = oracle.run(cfgs, p, seed=51, records=True)["records"]
    for precision, tol, bar in ((32, 1e-3, 0.99), (64, 1e-6, 0.999)):
        plan = spx.Plan(cfgs, p, precision=precision)
        rec = spx.records_to_numpy(plan.run(seed=51, records=True)["records"])
        if precision == 32:
            plan.set_launch(3, 64, 2, 8, 64)
            assert np.array_equal(rec, spx.records_to_numpy(plan.run(seed=51, records=True)["records"]))
        m = match_stats(rec, ref, tol)
        assert m["frac"] * m["n"] >= bar * m["n"] - 1, (precision, m)
