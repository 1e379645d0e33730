"""The bytes that the statistics count for the stored near-field tiles: the lanes of a 64 x 64 tile that
hold entries, alike for single vectors and blocks."""
import pytest
import torch

from paper_2501_17656_amd import H2Matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf,lanes", [(64 * 49, 64, 7), (64 * 33, 64, 5), (32 * 64, 64, 8), (32 * 98, 128, 7)])
def test_near_tile_bytes(n, leaf, lanes):
    gen = torch.Generator(device="cuda").manual_seed(n)
    pts = torch.rand((n, 2), dtype=torch.float64, device="cuda", generator=gen)
    X = torch.randn((n, 16), dtype=torch.float64, device="cuda", generator=gen)
    g = H2Matrix(pts, "exp", 0.2, 0.5, leaf, 0.7, 3)
    g.store_near()
    g.set_timing(True)
    g.matvec(X[:, 0].contiguous())
    g.matvec_multi(X)
    single, block = (g.kernel_stats(k) for k in ("near_gemv_fp64", "near_gemm16_fp64"))
    assert single["launches"] == block["launches"] == 1
    assert block["work"] == single["work"]
    assert single["work"] % (64 * lanes * lanes * 8) == 0
    # tiles read by a block product: all of them, and the off-diagonal ones for their column
    chunks = n // {7: 49, 5: 33, 8: 64}[lanes]
    tiles = single["work"] / (64 * lanes * lanes * 8)
    assert g.block_tuning()["near"]["tiles_read"] == 2 * tiles - chunks
    g.close()
