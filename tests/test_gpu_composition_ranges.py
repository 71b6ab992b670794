"""Composition map over the range that the entry point takes: from one row of many areas to many of one,
against plain FP64 arithmetic on the same inputs with the bar of the default sizes (2e-4 at.%); and
one long row costs as many short ones (8 times at most, where a block for it took 200)."""
import pytest

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


def _comp_inputs(B, J, K):
    g = torch.Generator(device="cuda").manual_seed(B + J + K)

    def u(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, device="cuda", generator=g)
    return [u(0.02, 0.2, K, J), u(0.5, 2, K), u(0, 0.2, K), u(20, 200, B, K), u(50, 200, K), u(8, 22, K), u(0.05, 0.15, K)]


@pytest.mark.parametrize("K", [1, 3, 4, 8, 9, 16])
@pytest.mark.parametrize("B, J", [(1, 255), (1, 256), (1, 257), (1, 5001), (2, 40000), (5, 2047), (7, 3), (130, 300), (511, 513), (4099, 31),
                                  (257, 1)])
def test_composition_of_many_areas(B, J, K):
    xs = _comp_inputs(B, J, K)
    c = spx.comp_forward(*xs)
    f, a, b, P, M, rho, fref = [x.double() for x in xs]
    y = ((a * P + b) * rho / (M * fref))[:, None, :] * f.t()[None]
    assert (c.double() - 100.0 * y / y.sum(dim=2, keepdim=True)).abs().max().item() < 2e-4


def test_one_row_of_many_areas_costs_as_many_rows():
    for K in (3, 4, 9):
        row, rows = _comp_inputs(1, 1_000_000, K), _comp_inputs(1000, 1000, K)
        t, t0 = _us(lambda: spx.comp_forward(*row)), _us(lambda: spx.comp_forward(*rows))
        say(f"K={K}: 1 x 1e6 areas {t:.0f} us, 1000 x 1000 {t0:.0f} us")
        assert t < 8 * t0
