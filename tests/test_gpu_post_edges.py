"""Post-processing kernels at the edges of their splits: composition map, its one-pass backward and the
one without scratch, squared distance, area average and covered area, against the oracle in float64.
Bars: those of the default sizes (2e-4 at.% forward, 2e-4 of the largest gradient, 1e-5 relative
distance, 1e-13 relative area average, covered areas bit for bit)."""
import ctypes

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

NAMES = ("f", "a", "b", "P", "M", "rho", "fref")


def _inputs(B, J, K):
    r = np.random.default_rng(B + 31 * J + 7 * K)
    f = r.uniform(0.02, 0.2, (K, J))
    return (f, r.uniform(0.5, 2, K), r.uniform(0, 0.2, K), r.uniform(20, 200, (B, K)), r.uniform(50, 200, K),
            r.uniform(8, 22, K), f.mean(axis=1))


def _cuda(*xs):
    return [torch.as_tensor(np.asarray(x), dtype=torch.float32, device="cuda").contiguous() for x in xs]


@pytest.mark.parametrize("B,J,K", [(1, 1, 2), (3, 63, 3), (4, 64, 4), (5, 65, 5), (1023, 342, 4), (9, 384, 8),
                                   (6, 385, 4), (2, 1536, 2), (3, 1537, 3), (7, 40, 9), (4200, 26, 1)])
def test_composition_and_backward(B, J, K):
    say(f"B={B} J={J} K={K}")
    xs = _inputs(B, J, K)
    dev = _cuda(*xs)
    c_ref = oracle.composition(*xs)
    c = spx.comp_forward(*dev)
    assert np.abs(c.cpu().numpy() - c_ref).max() < 2e-4
    # a gradient without the structure of a distance: every term counts
    gc = np.random.default_rng(B).normal(size=(B, J, K)).astype(np.float32)
    x64 = [torch.as_tensor(v, dtype=torch.float64).requires_grad_(True) for v in [t.cpu().numpy() for t in dev]]
    w = (x64[1] * x64[3] + x64[2]) * x64[5] / (x64[4] * x64[6])
    y = w[:, None, :] * x64[0].t()[None]
    (100.0 * y / y.sum(dim=2, keepdim=True) * torch.as_tensor(gc, dtype=torch.float64)).sum().backward()
    g = spx.comp_backward(*dev, torch.as_tensor(gc, device="cuda"))
    # the entry point without scratch, and c with an address that is only 4-byte aligned
    o = {n: torch.empty_like(t) for n, t in zip(NAMES, dev)}
    odd = torch.empty(B * J * K + 1, device="cuda")[1:]
    odd.copy_(torch.as_tensor(gc).reshape(-1))
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    spx.check(spx.lib().spx_comp_backward(*[p(t) for t in dev], p(odd), *[p(o[n]) for n in ("f", "a", "b", "P", "M", "rho", "fref")],
                                          B, J, K, st), "spx_comp_backward")
    h = spx.comp_backward(*dev, odd.view(B, J, K))
    for n, t in zip(NAMES, x64):
        # sums of gradients of either sign cancel: measured against what their terms amount to in the
        # element with the largest gradient, with K > 1 (one element alone has composition 100 and no gradient)
        scale = t.grad.abs().max().item() if K > 1 else 1e-2 * np.abs(gc).sum()
        for got in (g, o, h):
            assert np.abs(got[n].double().cpu().numpy() - t.grad.numpy()).max() <= 2e-4 * scale, n
    loss, gd = spx.comp_sqdist(c, torch.as_tensor(gc[0], device="cuda"), want_grad=True)
    d = c.double().cpu().numpy() - gc[:1]
    assert np.allclose(loss.cpu().numpy(), (d ** 2).sum(axis=(1, 2)), rtol=1e-5)
    assert np.allclose(gd.cpu().numpy(), 2 * d, rtol=1e-5, atol=1e-4)


@pytest.mark.parametrize("nu,nv,half", [(1, 1, 2.25), (7, 3, 2.25), (64, 65, 2.25), (200, 200, 0.1), (300, 40, 40.0)])
def test_area_average(nu, nv, half):
    say(f"{nu} x {nv} bins, half width {half}")
    g = si.Grid(nu=nu, nv=nv, half_u=50.0, half_v=45.0)
    prof = np.random.default_rng(nu).uniform(0.5, 1.5, (2, nv, nu))
    cen = np.array([[0.0, 0.0], [49.9, -44.9], [-60.0, 10.0], [12.34, -5.67], [50.0, 45.0]])
    got = spx.area_gather(torch.as_tensor(prof, device="cuda"), g, cen, half).cpu().numpy()
    for p in range(2):
        with np.errstate(invalid="ignore"):
            ref = oracle.area_gather(prof[p], g, cen, half)
        # a square that meets no bin has no mean (0 / 0 in the oracle): the library writes 0
        assert np.allclose(got[p], np.nan_to_num(ref, nan=0.0), rtol=1e-13, atol=0)


@pytest.mark.parametrize("J", [1, 2, 3, 63, 64, 65, 127, 128, 129, 257, 342, 513, 2048])
def test_covered_area(J):
    say(f"{J} compositions")
    r = np.random.default_rng(J)
    c = r.dirichlet((2.0, 3.0, 4.0), (3, J)).astype(np.float32) * 100
    c[1, :, 2] = c[1, :, 1]                        # collinear in the diagram
    c[2, J // 2:] = c[2, :J - J // 2]              # duplicates
    got = spx.hull_area(torch.as_tensor(c, device="cuda")).cpu().numpy()
    assert np.array_equal(got, np.array([oracle.hull_area_fraction(x) for x in c], dtype=np.float32))
