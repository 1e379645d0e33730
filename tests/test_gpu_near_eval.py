"""The evaluated near field at the edges of its tiles: leaf lengths around multiples of 8 and of the
64-row chunks, tasks split over waves and not, one to three dimensions, with per-point scale.  With a
tiny eta no block is far, so the product is the dense kernel matrix, formed here directly in FP64."""
import numpy as np
import pytest
import torch

from paper_2501_17656_amd import H2Matrix

pytestmark = pytest.mark.gpu

ELL = 0.3


def dense_product(pts, x, kernel, shift, scale=None, diag=None):
    y = torch.empty_like(x)
    for c in range(0, len(pts), 2048):
        r = torch.zeros(len(pts[c:c + 2048]), len(pts), dtype=torch.float64, device=x.device)
        for a in range(pts.shape[1]):
            r += (pts[c:c + 2048, None, a] - pts[None, :, a]) ** 2
        if kernel == "gauss":
            k = torch.exp(-r / (2 * ELL * ELL))
        elif kernel == "exp":
            k = torch.exp(-torch.sqrt(r) / ELL)
        else:
            z = 3.0 ** 0.5 * torch.sqrt(r) / ELL
            k = (1 + z) * torch.exp(-z)
        xs = x if scale is None else scale * x
        y[c:c + 2048] = k @ xs if scale is None else scale[c:c + 2048] * (k @ xs)
    return y + (shift * x if diag is None else diag * x)


# n, leaf size: the leaves hold n / 2^L points, rounded up or down
SIZES = [(9, 16), (17, 32), (63, 64), (64, 64), (65, 128), (200, 256), (256, 256), (8 * 33, 40), (8 * 48 + 3, 64),
         (8 * 64, 64), (4 * 65 + 1, 80), (4 * 98, 128), (4 * 128 - 1, 128), (2 * 231 + 1, 256),
         (256 * 17 + 5, 20), (256 * 66 - 9, 70)]       # more than 12288 pairs: whole leaves per wave


@pytest.mark.parametrize("n,leaf", SIZES)
@pytest.mark.parametrize("dim,kernel", [(1, "exp"), (2, "gauss"), (3, "matern32")])
def test_near(n, leaf, dim, kernel):
    rng = np.random.default_rng(n + dim)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    pts, x = dev(rng.random((n, dim))), dev(rng.standard_normal(n))
    s, d = dev(0.5 + rng.random(n)), dev(1.0 + rng.random(n))
    for kw in ({}, {"scale": s, "diag": d}, {"scale": s}):
        g = H2Matrix(pts, kernel, ELL, 0.25, leaf, 1e-9, 2, **kw)
        y = g.matvec(x)
        want = dense_product(pts, x, kernel, 0.25, **kw)
        # sums of n products, each within a few roundings of its exact value
        bound = 16 * n ** 0.5 * 2.0 ** -53 * float(x.norm()) * n ** 0.5 * (2.25 if kw else 1.0)
        assert float((y - want).norm()) <= bound
        g.close()


@pytest.mark.parametrize("n,leaf", [(8 * 48 + 3, 64), (4 * 98, 128), (256 * 17 + 5, 20)])
def test_near_fp32(n, leaf):
    rng = np.random.default_rng(n)
    pts, x = torch.from_numpy(rng.random((n, 3))).cuda(), torch.from_numpy(rng.standard_normal(n)).cuda()
    g = H2Matrix(pts, "exp", ELL, 1.0, leaf, 1e-9, 2)
    g.setup(["fp64", "fp32"])
    y = g.level_apply(1, x, precision="fp32")
    want = dense_product(pts, x, "exp", 1.0)
    assert float((y - want).norm()) <= 16 * n * 2.0 ** -24 * float(x.norm()), float((y - want).norm())
    g.close()


@pytest.mark.parametrize("dim,kernel", [(2, "exp"), (3, "matern32"), (3, "gauss")])
@pytest.mark.parametrize("unit", [1.0, 1e10, 1e-16])
def test_near_far_out(unit, dim, kernel):
    """Distances of up to 1e10 length scales (no entry but the diagonal counts) and coordinates whose
    squares leave FP32's normal range, in FP64 and FP32."""
    n = 4 * 98
    if kernel == "gauss" and unit < 1:
        pytest.skip("1 / (2 l^2) is not an FP32 number")
    rng = np.random.default_rng(n)
    pts, x = torch.from_numpy(rng.random((n, dim))).cuda(), torch.from_numpy(rng.standard_normal(n)).cuda()
    g = H2Matrix(unit * pts, kernel, ELL * min(unit, 1.0), 1.0, 128, 1e-9, 2)
    g.setup(["fp64", "fp32"])
    want = dense_product(max(unit, 1.0) * pts, x, kernel, 1.0)
    for y, eps in ((g.matvec(x), 2.0 ** -53), (g.level_apply(1, x, precision="fp32"), 2.0 ** -24)):
        assert float((y - want).norm()) <= 16 * n * eps * float(x.norm())
    g.close()


@pytest.mark.parametrize("n,dim,m,leaf,kernel", [
    (3000, 1, 20, 40, "exp"), (5000, 2, 5, 60, "gauss"), (4099, 2, 6, 80, "matern32"), (6000, 2, 8, 100, "exp"),
    (6001, 3, 3, 50, "laplace"), (8000, 3, 4, 130, "matern32"), (20000, 3, 4, 90, "gauss")])
def test_near_with_couplings(n, dim, m, leaf, kernel):
    """One launch for close pairs and couplings gives what two give, bit for bit (kernel timing asks for
    two): tiles of 32 and 64, full and not, leaves on both sides of 64 points, scaled and not."""
    rng = np.random.default_rng(n)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    pts, x = dev(rng.random((n, dim))), dev(rng.standard_normal(n))
    scaled = {"scale": dev(0.5 + rng.random(n)), "diag": dev(1.0 + rng.random(n))}
    for kw in ({}, scaled):
        g = H2Matrix(pts, kernel, ELL, 0.0 if kernel == "laplace" else 1.0, leaf, 0.7, m, **kw)
        y = g.matvec(x)
        g.set_timing(True)
        assert torch.equal(y, g.matvec(x))
        assert g.kernel_stats("gemv_fp64")["launches"] == 1 and g.kernel_stats("near_fp64")["launches"] == 1
        g.set_timing(False)
        assert torch.equal(y, g.matvec(x))
        g.close()
