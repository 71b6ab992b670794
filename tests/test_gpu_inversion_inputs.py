"""Libraries that the inversion's kernels have to take as they are: compositions far from the range of at.%
(other units, values not normalised), whose covered areas are the oracle's bit for bit (float64 value
rounded to float), and areas that no atom reached, which have no composition."""
import numpy as np
import pytest

import oracle
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("J", [64, 342, 2048])
@pytest.mark.parametrize("place, size", [(0.0, 1.0), (40.0, 10.0), (0.0, 300.0), (-200.0, 100.0), (1e5, 100.0), (9e5, 10.0), (988875.0, 7.5),
                                         (0.0, 1e-3), (0.0, 1e30)])
def test_covered_area_anywhere(J, place, size):
    say(f"{J} compositions around {place}, spread {size}")
    r = np.random.default_rng(J)
    t = r.uniform(0, 2 * np.pi, (3, J))
    rad = np.sqrt(r.uniform(0, 1, (3, J)))
    rad[1] = r.uniform(0.999, 1.0, J)               # a rim: most points near an edge of the hull
    c = np.zeros((3, J, 3), dtype=np.float32)
    c[:, :, 1] = place + size * rad * np.cos(t)
    c[:, :, 2] = place + size * rad * np.sin(t)
    got = spx.hull_area(torch.as_tensor(c, device="cuda")).cpu().numpy()
    with np.errstate(over="ignore"):
        ref = np.array([oracle.hull_area_fraction(x) for x in c], dtype=np.float32)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("J", [8, 342])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_covered_area_of_an_empty_area(J, bad):
    # an area that no atom reached has no composition: neither has the library a covered area
    r = np.random.default_rng(J)
    c = r.dirichlet((2.0, 3.0, 4.0), (3, J)).astype(np.float32) * 100
    c[0, 0] = c[1, J // 2] = c[2, J - 1] = bad
    assert not np.isfinite(spx.hull_area(torch.as_tensor(c, device="cuda")).cpu().numpy()).any()


def test_zero_rates_give_nan_compositions():
    # areas and elements without atoms: 0 / 0 in the map as in the definition, and only there
    r = np.random.default_rng(2)
    for K in (3, 4, 9):
        f = r.uniform(0.02, 0.2, (K, 70))
        f[:, 5] = f[:, 69] = 0.0
        f[0, 7] = 0.0
        xs = [f, r.uniform(0.5, 2, K), r.uniform(0, 0.2, K), r.uniform(20, 200, (2, K)), r.uniform(50, 200, K),
              r.uniform(8, 22, K), np.full(K, 0.1)]
        c = spx.comp_forward(*[torch.as_tensor(x, dtype=torch.float32, device="cuda") for x in xs])
        ok = np.isfinite(c.cpu().numpy())
        assert not ok[:, [5, 69]].any() and ok[:, [j for j in range(70) if j not in (5, 69)]].all()
        assert (c[:, 7, 0] == 0).all()
        loss, gc = spx.comp_sqdist(c, torch.zeros(70, K, device="cuda"), want_grad=True)
        assert torch.isnan(loss).all() and torch.equal(torch.isnan(gc), torch.isnan(c))
