"""The stored near field at the edges of its chunks: leaves cut into one to four chunks of equal length,
full ones and ones that fill their 64 x 64 tiles only in part.  Single vectors and blocks, against the
product with the close blocks evaluated."""
import pytest
import torch

from paper_2501_17656_amd import H2Matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(9, 16), (63, 64), (64, 64), (65, 128), (129, 256), (193, 256), (256, 256),
                                    (8 * 49 + 3, 64), (4 * 98, 128), (16 * 57 - 1, 64), (32 * 128, 128), (64 * 33, 40)])
def test_chunks(n, leaf):
    gen = torch.Generator(device="cuda").manual_seed(n)
    pts = torch.rand((n, 2), dtype=torch.float64, device="cuda", generator=gen)
    X = torch.randn((n, 16), dtype=torch.float64, device="cuda", generator=gen)
    g = H2Matrix(pts, "exp", 0.2, 0.5, leaf, 0.7, 3)
    want = torch.stack([g.matvec(X[:, k].contiguous()) for k in (0, 15)], 1)
    blocks = [g.matvec_multi(X)]
    g.store_near()
    y = torch.stack([g.matvec(X[:, k].contiguous()) for k in (0, 15)], 1)
    blocks.append(g.matvec_multi(X))
    bound = 1e-14 * n ** 0.5 * float(want.norm())       # sums of n products each
    assert float((y - want).norm()) <= bound
    for Y in blocks:
        assert float((Y[:, [0, 15]] - want).norm()) <= bound
    g.close()
