"""Post-processing calls of more rows than one launch has blocks for: every row is done, the last as the
first (2e-4 at.% and 2e-4 of the largest gradient, the bars of the default sizes)."""
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402

BLOCKS = (2**32 - 1) // 256          # blocks of 256 threads in a launch


def _comp_inputs(B, J, K):
    g = torch.Generator(device="cuda").manual_seed(B + J + K)

    def u(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, device="cuda", generator=g)
    return [u(0.02, 0.2, K, J), u(0.5, 2, K), u(0, 0.2, K), u(20, 200, B, K), u(50, 200, K), u(8, 22, K), u(0.05, 0.15, K)]


def test_composition():
    B = (1 << 30) + 4097
    say(f"{B} rows of one area and one element")
    xs = _comp_inputs(1, 1, 1)
    xs[3] = torch.full((B, 1), 50.0, device="cuda")
    c = spx.comp_forward(*xs)
    assert float((c - 100.0).abs_().max()) < 2e-4


def test_distance():
    B = 4 * BLOCKS + 5
    say(f"{B} rows of one value")
    c = torch.arange(B, dtype=torch.float32, device="cuda").remainder_(977.0).view(B, 1, 1)
    loss, gc = spx.comp_sqdist(c, torch.full((1, 1), 2.0, device="cuda"), want_grad=True)
    d = c - 2.0                       # whole numbers: exact
    assert torch.equal(gc, 2.0 * d) and torch.equal(loss, (d * d).view(B))


def test_backward_without_scratch():
    B, K = BLOCKS + 3, 9
    say(f"{B} rows of {K} elements, one area")
    xs = _comp_inputs(B, 1, K)
    gc = torch.rand(B, 1, K, device="cuda")
    got = spx.comp_backward(*xs, gc)["P"][-1000:]
    f, a, b, P, M, rho, fref = [x.double() for x in xs[:3] + [xs[3][-1000:]] + xs[4:]]
    P.requires_grad_(True)
    y = (a * P + b) * rho / (M * fref) * f[:, 0]
    (100.0 * y / y.sum(dim=1, keepdim=True) * gc[-1000:, 0].double()).sum().backward()
    assert (got.double() - P.grad).abs().max().item() <= 2e-4 * P.grad.abs().max().item()


def test_covered_area():
    B = BLOCKS + 2
    say(f"{B} libraries of three areas")
    c = torch.zeros(B, 3, 3, device="cuda")
    c[:, [0, 1, 2], [0, 1, 2]] = 100.0
    assert (spx.hull_area(c) == 1.0).all()


def test_sweep_composition():
    T = BLOCKS + 2
    say(f"{T} sweep points of one area and one element")
    one = [torch.ones(1, dtype=torch.float64, device="cuda") for _ in range(5)]
    assert (spx.sweep_composition(torch.full((T, 1, 1), 0.5, dtype=torch.float64, device="cuda"), *one) == 100.0).all()


def test_composition_of_the_most_areas():
    J = 2**31 - 1
    say(f"one row of {J} areas")
    xs = _comp_inputs(1, 1, 1)
    xs[0] = torch.full((1, J), 0.25, device="cuda")
    c = spx.comp_forward(*xs)
    assert float((c - 100.0).abs_().max()) < 2e-4
