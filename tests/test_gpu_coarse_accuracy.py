"""The direct solve of the coarsest operator on ill-conditioned matrices: its residual is that of
substitution with the Cholesky factor.  With a tiny eta there are no far blocks, so one cycle is the
direct solve of the whole matrix, in the order of the tree; residuals are formed on the host in
extended precision."""
import numpy as np
import pytest
import torch
from scipy.linalg import cho_factor, cho_solve

from paper_2501_17656_amd import H2Matrix
from paper_2501_17656_amd.h2mg import Plan

pytestmark = pytest.mark.gpu


def kernel_matrix(pts, ell, shift):
    r2 = ((pts[:, None] - pts[None]) ** 2).sum(2)
    return np.exp(-r2 / (2 * ell * ell)) + shift * np.eye(len(pts))


# condition numbers of about 1e3 to 1e4, 1e7 to 1e8, 4e11 to 4e12, and 4e13 to 4e14
@pytest.mark.parametrize("ell,shift", [(0.1, 1e-2), (0.1, 1e-6), (0.2, 1e-10), (0.2, 1e-12)])
@pytest.mark.parametrize("n", [200, 577, 1000, 2048])
def test_residual_is_that_of_substitution(n, ell, shift):
    rng = np.random.default_rng(n)
    pts, B = rng.random((n, 2)), rng.standard_normal((n, 16))
    pts = np.ascontiguousarray(pts[Plan(pts, 64, 1e-9, 3).perm()])   # the tree's order: its own permutation
    assert (Plan(pts, 64, 1e-9, 3).perm() == np.arange(n)).all()
    A = kernel_matrix(pts, ell, shift)
    factor, wide = cho_factor(A, lower=True), A.astype(np.longdouble)

    def residuals(X):
        return np.linalg.norm((B[:, :X.shape[1]] - wide @ X).astype(np.float64), axis=0)
    # both are a few roundings away from a backward stable solve with the same factor; the order of
    # the sums differs, and so does the luck of the single columns: their mean, within a factor of 4
    want = residuals(cho_solve(factor, B)).mean()
    g = H2Matrix(torch.from_numpy(pts).cuda(), "gauss", ell, shift, 64, 1e-9, 3)
    g.setup(["fp64"])
    b = torch.from_numpy(B).cuda()
    zero = torch.zeros_like(b[:, 0])
    single = torch.stack([g.vcycle(zero, b[:, k].contiguous()) for k in range(16)], 1)
    block, _ = g.solve_multi(b, rtol=1e-30, max_cycles=1, raise_on_error=False)
    assert residuals(single.cpu().numpy()).mean() <= 4 * want
    assert residuals(block.cpu().numpy()).mean() <= 4 * want
    g.close()
