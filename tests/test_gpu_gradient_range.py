"""Gradients of the composition map where rates or gradients are very small or large (other units, scaled
losses): a product of both may leave the range of FP32 though the gradients do not (2e-4 of the largest
gradient, the bar of the default sizes)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("rate, grad", [(1.0, 1.0), (1e-20, 1e-20), (1e-25, 1e-10), (1e18, 1e22), (1e-12, 1e-30), (3e-38, 1e-10)])
@pytest.mark.parametrize("J, K", [(342, 4), (400, 3), (50, 8), (1600, 2)])
def test_backward(J, K, rate, grad):
    g = torch.Generator(device="cuda").manual_seed(J)

    def u(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, device="cuda", generator=g)
    B = 9
    xs = [rate * u(0.02, 0.2, K, J), u(0.5, 2, K), u(0, 0.2, K), u(20, 200, B, K), u(50, 200, K), u(8, 22, K), u(0.5, 1.5, K)]
    gc = grad * torch.randn(B, J, K, device="cuda", generator=g)
    got = spx.comp_backward(*xs, gc)
    x64 = [x.double().requires_grad_(True) for x in xs]
    f, a, b, P, M, rho, fref = x64
    y = ((a * P + b) * rho / (M * fref))[:, None, :] * f.t()[None]
    (100.0 * y / y.sum(dim=2, keepdim=True) * gc.double()).sum().backward()
    for name, x in zip(("f", "a", "b", "P", "M", "rho", "fref"), x64):
        assert (got[name].double() - x.grad).abs().max().item() <= 2e-4 * x.grad.abs().max().item(), name
