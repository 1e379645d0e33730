"""The direct solve of the coarsest operator at the edges of its blocks: the inverse of the Cholesky
factor (orders around multiples of 64, and up to 8192), and substitution above.  With a tiny eta there
are no far blocks, so one cycle is the direct solve of the whole matrix."""
import numpy as np
import pytest
import torch

from paper_2501_17656_amd import H2Matrix

pytestmark = pytest.mark.gpu

ELL, SHIFT = 0.02, 1.0


def matrix(pts):
    r2 = sum((pts[:, None, a] - pts[None, :, a]) ** 2 for a in range(2))
    return torch.exp(-r2 / (2 * ELL * ELL)) + SHIFT * torch.eye(len(pts), dtype=pts.dtype, device=pts.device)


@pytest.mark.parametrize("n", [9, 63, 64, 65, 100, 128, 129, 200, 256, 300, 577, 1000, 2049, 8200])
def test_direct_solve(n):
    rng = np.random.default_rng(n)
    pts = torch.from_numpy(rng.random((n, 2))).cuda()
    b = torch.from_numpy(rng.standard_normal((n, 16))).cuda()
    g = H2Matrix(pts, "gauss", ELL, SHIFT, 64 if n > 16 else 16, 1e-9, 3)
    g.setup(["fp64", "fp32"])
    A = matrix(pts)
    # the norm (at most the largest row sum) over the smallest eigenvalue (at least the shift)
    kappa = float(A.sum(1).max()) / SHIFT
    bound = 4 * kappa * n ** 0.5 * 2.0 ** -53

    def off(x, c):
        return float((A @ x - b[:, c]).norm() / b[:, c].norm())
    x = g.vcycle(torch.zeros_like(b[:, 0]), b[:, 0].contiguous())
    assert off(x, 0) <= bound
    X, info = g.solve_multi(b, rtol=1e-11)
    assert max(off(X[:, c], c) for c in range(16)) <= 1e-11 + bound and info["cycles"] == 1
    # FP32 vectors around the FP64 factor: one step is good to FP32, three are good to 1e-11
    x, info = g.solve(b[:, 1].contiguous(), rtol=1e-11, precision="fp32")
    assert off(x, 1) <= 1e-11 + bound and info["cycles"] <= 4
    X, info = g.solve_multi(b, rtol=1e-11, precision="fp32")
    assert max(off(X[:, c], c) for c in range(16)) <= 1e-11 + bound and info["cycles"] <= 4
    g.close()
