"""Roundings and range of the kernel entries.  One leaf and no far block, so the product with a unit
vector is a column of the kernel matrix: point 0 at the origin, the others on an axis."""
import numpy as np
import pytest
import torch

from paper_2501_17656_amd import H2Matrix

pytestmark = pytest.mark.gpu

LOG2E = np.float64(1.4426950408889634)


def column(r, kernel, ell, path="fp64", derivative="value", diag=None):
    """Entries k(r) as a product with the unit vector of point 0 gives them (r[0] = 0: with the diagonal)."""
    pts = np.zeros((r.size, 3))
    pts[:, 0] = r
    kw = {"diag": torch.full((r.size,), diag, dtype=torch.float64, device="cuda")} if diag else {}
    shift = 1.0 if derivative == "value" and not diag else 0.0
    g = H2Matrix(torch.from_numpy(pts).cuda(), kernel, ell, shift, 256, 0.7, 3, derivative=derivative, **kw)
    e0 = torch.zeros(r.size, dtype=torch.float64, device="cuda")
    e0[0] = 1.0
    if path == "fp64":
        k = g.matvec(e0)
    elif path == "fp64_block":
        k = g.matvec_multi(torch.stack([e0, 2 * e0], 1).contiguous())[:, 0]
    else:
        g.setup(["fp64", "fp32"])
        k = g.level_apply(1, e0, precision="fp32")
    g.close()
    return k.cpu().numpy()


def exponent(kernel, r, ell):
    """The exponent z of the kernel, and what a relative error of z is in the entry."""
    r, ell = r.astype(np.longdouble), np.longdouble(ell)
    if kernel == "gauss":
        z = r * r / (2 * ell * ell)
    else:
        z = r / ell * (np.sqrt(np.longdouble(3)) if kernel == "matern32" else 1)
    return z, (z * z / (1 + z) if kernel == "matern32" else z)


def value(kernel, z):
    return (1 + z) * np.exp(-z) if kernel == "matern32" else np.exp(-z)


@pytest.mark.parametrize("path", ["fp64", "fp32", "fp64_block"])
@pytest.mark.parametrize("kernel", ["exp", "gauss", "matern32"])
def test_exponent_coefficient_is_rounded_once(kernel, path):
    """The factor of the distance in the exponent is off by one rounding at most (u), also for length
    scales for which the product of a rounded 1 / l (or 1 / (2 l^2)) with a rounded log2(e) is off by
    nearly two and more.  The other roundings of an entry have no sign: over 255 entries their mean is
    below a quarter of u (each is at most u, the exponential's twice that over z >= 10)."""
    ft, u = (np.float32, 2.0 ** -24) if path == "fp32" else (np.float64, 2.0 ** -53)
    ells = 0.1 * (1 + 1e-3 * np.arange(400))
    if kernel == "gauss":
        twice = ft(1.0 / (2.0 * ells * ells)) * ft(LOG2E)
        once = np.log2(np.exp(np.longdouble(1))) / (2 * ells.astype(np.longdouble) ** 2)
    else:
        c = np.sqrt(np.longdouble(3)) if kernel == "matern32" else np.longdouble(1)
        twice = ft(1.0 / ells) * ft(c.astype(np.float64) * LOG2E)
        once = c * np.log2(np.exp(np.longdouble(1))) / ells.astype(np.longdouble)
    off = np.abs(twice / once - 1).astype(np.float64)
    for ell in ells[np.argsort(off)[-3:]]:
        z0 = np.geomspace(10, 40, 255)
        s = {"gauss": np.sqrt(2 * z0), "exp": z0, "matern32": z0 / 3.0 ** 0.5}[kernel]
        r = np.concatenate([[0.0], ell * s])
        z, sens = exponent(kernel, r[1:], ell)
        err = (column(r, kernel, ell, path)[1:] / value(kernel, z) - 1) / sens
        assert abs(float(err.mean())) <= 1.25 * u, (ell, float(err.mean()) / u)


@pytest.mark.parametrize("kernel", ["exp", "gauss", "matern32"])
def test_fp32_entries_below_the_normal_range(kernel):
    """FP32 entries underflow gradually: off by the roundings of the exponent (2 ulp of z) and of the
    entry, and by one unit of the subnormal numbers in the exponential."""
    ell, z0 = 0.1, np.linspace(87.5, 102.0, 255)
    s = {"gauss": np.sqrt(2 * z0), "exp": z0, "matern32": z0 / 3.0 ** 0.5}[kernel]
    r = np.concatenate([[0.0], ell * s])
    z, _ = exponent(kernel, r[1:], ell)
    want = value(kernel, z)
    err = np.abs(column(r, kernel, ell, "fp32")[1:] - want)
    assert (err <= (6 + 4 * z) * 2.0 ** -24 * want + (1 + z) * 2.0 ** -149).all()


@pytest.mark.parametrize("path", ["fp64", "fp64_block"])
@pytest.mark.parametrize("kernel", ["exp", "matern32"])
@pytest.mark.parametrize("ell", [1e-140, 1e-150])
def test_tiny_length_scales(ell, kernel, path):
    """Coincident points have the kernel's value at 0, and distances whose squares are near the end of the
    normal range their own root: within the roundings of the exponent (2 ulp of z) and the entry."""
    r = np.concatenate([[0.0, 0.0], ell * np.geomspace(1e-3, 30.0, 60)])
    z, _ = exponent(kernel, r, ell)
    want = value(kernel, z)
    k = column(r, kernel, ell, path)
    assert k[1] == 1.0
    assert (np.abs(k[1:] - want[1:]) <= (6 + 4 * z[1:]) * 2.0 ** -53 * want[1:]).all()


@pytest.mark.parametrize("path", ["fp64", "fp32", "fp64_block"])
def test_laplace_entries_over_the_whole_range(path):
    """1 / (4 pi r) also where r^2 is subnormal in FP32, and 0 where it is no finite number."""
    r = np.concatenate([[0.0], np.geomspace(1e-20, 1e-17, 20), np.geomspace(1e-10, 1e10, 20), [1e25, 1e160]])
    k = column(r, "laplace", 1.0, path, diag=1e23)[1:]
    r = r[1:]
    if path == "fp32":
        # r^2 has an absolute error of 2^-150 there, besides 4 roundings
        bound = (2.0 ** -22 + 0.5 * 2.0 ** -150 / r / r) / (4 * np.pi * r)
        zero = r >= 1e25
    else:
        bound, zero = 2.0 ** -50 / (4 * np.pi * r), r >= 1e160
    assert (k[zero] == 0.0).all()
    assert (np.abs(k - 1 / (4 * np.pi * r)) <= bound)[~zero].all()


@pytest.mark.parametrize("kernel", ["exp", "gauss", "matern32"])
@pytest.mark.parametrize("derivative", ["dl", "g"])
def test_derivative_entries_over_the_whole_range(derivative, kernel):
    """Tiny length scales, whose inverse cube is no finite number, and distances whose squares are none:
    the exact value within the roundings of the exponent (2 ulp of z) and of the factors, 0 where it
    underflows."""
    for ell, r in ((1e-110, 1e-110 * np.geomspace(1e-2, 20.0, 60)), (0.1, np.append(np.geomspace(0.01, 1.0, 40), 1e160))):
        z, _ = exponent(kernel, r, ell)
        x, L, e = r.astype(np.longdouble), np.longdouble(ell), np.exp(-z)
        if derivative == "dl":
            want = {"exp": x / L ** 2, "gauss": x * x / L ** 3, "matern32": z * z / L}[kernel] * e
        else:
            want = {"exp": -1 / (L * x), "gauss": -1 / L ** 2, "matern32": -3 / L ** 2}[kernel] * e
        k = column(np.concatenate([[0.0], r]), kernel, ell, "fp64", derivative)[1:]
        big = r > 1e100
        assert (k[big] == 0.0).all()
        err = np.abs(k - want) <= (12 + 4 * np.minimum(z, 1e3)) * 2.0 ** -53 * np.abs(want)
        assert err[~big].all(), (ell, k[~big], want[~big])
