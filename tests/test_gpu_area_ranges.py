"""Area averages over the range that the entry point takes: squares of one bin to whole profiles, one square
to tens of millions, against plain FP64 arithmetic on the same inputs (1e-11 relative: sums of up to
4e4 terms of one sign); and small squares do not cost as large ones (8 times the time of the same
number of bins at most, where a wave per square took 49)."""
import pytest

import sputter_inputs as si
from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


def _us(fn):
    """Least time of a call among others, in us."""
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        fn()
        a.record()
        for _ in range(10):
            fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100.0)
    return best


def _area64(prof, grid, cen, hw):
    """Overlap-weighted means of [n, nv, nu] profiles over the squares, on the device in float64."""
    def overlap(c, half, n):
        d = 2.0 * half / n
        lo = -half + d * torch.arange(n, dtype=torch.float64, device="cuda")
        return torch.clamp(torch.minimum(lo + d, c[:, None] + hw) - torch.maximum(lo, c[:, None] - hw), min=0.0)
    ou, ov = overlap(cen[:, 0], grid.half_u, grid.nu), overlap(cen[:, 1], grid.half_v, grid.nv)
    s = torch.stack([((ov @ p) * ou).sum(dim=1) for p in prof])
    return torch.nan_to_num(s / (ov.sum(dim=1) * ou.sum(dim=1)), nan=0.0)


@pytest.mark.parametrize("n_prof, nu, nv, n_areas, hw", [
    (1, 50, 50, 342, 2.25), (3, 200, 200, 342, 2.25), (7, 50, 50, 5000, 0.4), (64, 50, 50, 2000, 1.0), (300, 20, 33, 700, 2.25),
    (2, 200, 150, 30000, 0.25), (2, 64, 200, 1, 60.0), (40, 200, 200, 342, 8.0), (5, 3, 300, 999, 4.0)])
def test_area_average_of_many_squares(n_prof, nu, nv, n_areas, hw):
    g = si.Grid(nu=nu, nv=nv, half_u=50.0, half_v=45.0)
    gen = torch.Generator(device="cuda").manual_seed(n_areas)
    prof = 0.5 + torch.rand(n_prof, nv, nu, dtype=torch.float64, device="cuda", generator=gen)
    cen = 110.0 * torch.rand(n_areas, 2, dtype=torch.float64, device="cuda", generator=gen) - 55.0
    got = spx.area_gather(prof, g, cen, hw)
    assert torch.allclose(got, _area64(prof, g, cen, hw), rtol=1e-11, atol=0)


def test_small_squares_cost_a_fraction_of_large_ones():
    # 4e6 squares of about 4 bins, and 4e4 of about 400: the same number of bins
    g = si.Grid(nu=50, nv=50, half_u=50.0, half_v=50.0)
    big = si.Grid(nu=500, nv=500, half_u=50.0, half_v=50.0)
    gen = torch.Generator(device="cuda").manual_seed(5)
    cen = 90.0 * torch.rand(2000, 2, dtype=torch.float64, device="cuda", generator=gen) - 45.0
    many = torch.rand(2000, 50, 50, dtype=torch.float64, device="cuda", generator=gen)
    few = torch.rand(20, 500, 500, dtype=torch.float64, device="cuda", generator=gen)
    t, t0 = _us(lambda: spx.area_gather(many, g, cen, 0.9)), _us(lambda: spx.area_gather(few, big, cen, 2.0))
    say(f"4e6 squares of 4 bins {t:.0f} us, 4e4 of 400 {t0:.0f} us")
    assert t < 8 * t0


def test_seventy_million_squares():
    say("7e7 squares of one bin")
    g = si.Grid(nu=1, nv=1, half_u=50.0, half_v=50.0)
    prof = torch.arange(1000, dtype=torch.float64, device="cuda").view(1000, 1, 1)
    got = spx.area_gather(prof, g, torch.zeros(70_000, 2, dtype=torch.float64, device="cuda"), 2.0)
    assert torch.equal(got, prof.view(1000, 1).expand(1000, 70_000))
