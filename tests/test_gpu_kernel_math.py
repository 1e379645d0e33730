"""Close entries over the whole range of distances: coincident points, separations whose squares
underflow, ordinary ones, and exponentials that underflow.  One leaf and no far block, so the
product with a unit vector is a column of the kernel matrix."""
import numpy as np
import pytest
import torch

from paper_2501_17656_amd import H2Matrix

pytestmark = pytest.mark.gpu

ELL = 0.1


def distances():
    return np.concatenate([[0.0, 0.0, 1e-170, 1e-150, 1e-100, 1e-20, 1e-8], ELL * np.geomspace(1e-6, 700.0, 50),
                           [ELL * 2000.0, ELL * 1e12, 1e100, 1e160]])


def exact(kernel, r):
    r = r.astype(np.longdouble)
    with np.errstate(over="ignore", under="ignore"):
        if kernel == "gauss":
            z = r * r / (2 * np.longdouble(ELL) ** 2)
            return np.exp(-z), z
        if kernel == "exp":
            z = r / np.longdouble(ELL)
            return np.exp(-z), z
        z = np.sqrt(np.longdouble(3)) * r / np.longdouble(ELL)
        return (1 + z) * np.exp(-z), z


@pytest.mark.parametrize("path", ["fp64", "fp32", "fp64_block"])
@pytest.mark.parametrize("kernel", ["exp", "gauss", "matern32"])
def test_entries(kernel, path):
    r = distances()
    pts = np.zeros((r.size, 3))
    pts[:, 0] = r
    g = H2Matrix(torch.from_numpy(pts).cuda(), kernel, ELL, 1.0, 64, 0.7, 3)
    e0 = torch.zeros(r.size, dtype=torch.float64, device="cuda")
    e0[0] = 1.0
    if path == "fp64":
        k = g.matvec(e0)
    elif path == "fp64_block":
        k = g.matvec_multi(torch.stack([e0, 2 * e0], 1).contiguous())[:, 0]
    else:
        g.setup(["fp64", "fp32"])
        k = g.level_apply(1, e0, precision="fp32")
    k = k.cpu().numpy()
    k[0] -= 1.0                          # the shift, which makes the matrix positive definite
    want, z = exact(kernel, r)
    # the exponent's roundings (constant, product, root: at most 2 ulp of z) and those of the
    # exponential, the polynomial factor and the sums (at most 6 ulp); results below the smallest
    # normal number may be flushed
    u, tiny = (2.0 ** -24, 2.0 ** -126) if path == "fp32" else (2.0 ** -53, 2.0 ** -1022)
    err = np.abs(k - want).astype(np.float64)
    bound = np.where(z < 1e6, (6 + 4 * np.minimum(z, 1e6)) * u, 0.0).astype(np.float64) * want.astype(np.float64) + tiny
    bad = ~(err <= bound)
    assert not bad.any(), [(r[i], k[i], float(want[i])) for i in np.nonzero(bad)[0]]
    assert (k[:6] == 1.0).all()          # r = 0 and separations that change nothing: exactly 1
    g.close()
