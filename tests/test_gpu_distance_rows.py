"""Squared distances on both sides of the number of rows from which each is a wave's and not a block's, against
plain FP64 arithmetic on the same inputs (1e-5 relative, the bar of the default sizes), and the same
bits on both sides."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2411_14413_amd as spx  # noqa: E402


@pytest.mark.parametrize("B, n", [(1, 5), (4096, 20001), (8191, 1369), (8192, 1369), (8193, 8193)])
def test_distance_of_long_rows(B, n):
    g = torch.Generator(device="cuda").manual_seed(n)
    c, t = torch.randn(B, n, 1, device="cuda", generator=g), torch.randn(n, 1, device="cuda", generator=g)
    loss, gc = spx.comp_sqdist(c, t, want_grad=True)
    d = c.double() - t.double()
    assert torch.allclose(loss.double(), (d * d).sum(dim=(1, 2)), rtol=1e-5)
    assert torch.allclose(gc.double(), 2 * d, rtol=1e-5, atol=1e-4)


@pytest.mark.parametrize("n", [1, 63, 256, 1368, 4099])
def test_a_row_alone_has_the_bits_of_a_row_among_many(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    c, t = torch.randn(8192, n, 1, device="cuda", generator=g), torch.randn(n, 1, device="cuda", generator=g)
    many = spx.comp_sqdist(c, t)
    assert torch.equal(spx.comp_sqdist(c[:100].contiguous(), t), many[:100])
