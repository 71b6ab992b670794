"""Table build at sizes around the edges of its kernels (quads of lanes, blocks of 64 angles, one block
per energy node): the oracle's quadrature within 1e-10, the bar of the default table, whose range of
energies these share, and the FP32 runs on such a table those of the oracle's."""
import math

import numpy as np
import pytest

import oracle
import sputter_inputs as si
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("ne,ns,theta_min", [(2, 2, 0.1), (3, 65, 0.1), (65, 3, 0.05), (257, 2, 0.1), (17, 130, 0.2)])
def test_table_sizes_match_oracle(ne, ns, theta_min):
    say(f"table {ne} x {ns}, theta_min {theta_min}")
    p = si.Params(table_ne=ne, table_ns=ns, theta_min=theta_min)
    th, bm = spx.Plan([si.single_ni(0.5, 10)], p).table()
    oth, obm = oracle.table(p)
    assert th.shape == (ne, ns) and bm.shape == (ne,)
    assert np.abs(th.ravel() - oth).max() < 1e-10
    assert np.abs(bm / obm - 1).max() < 1e-10
    assert np.all(th[:, 0] == math.pi)
