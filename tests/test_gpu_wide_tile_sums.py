"""Dense float32 sums of the widest tiles of the channel-last kernel (csrc/cb_fused_cl.h) against float64: a sum is rounded about once per 32 products, where one chain of
six products for each rounds it six times."""
import pytest
import torch

from test_gpu_wide_tiles import TILES, conv64, full_update, generator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", TILES)
def test_dense_sums(tile):
    """Weights of either sign: partial sums grow like a random walk of G = K / 32 steps, a rounding of each errs by 2^-24 / sqrt(3) of it at most: sqrt(G / 6) * 2^-24 of the sum,
    half as much again allowed, and 2^-24 for the result.  (Six roundings a group: sqrt(G) * 2^-24.)"""
    what, ci, co, k, H, W = tile
    print("dense sums", tile, flush=True)
    g = generator(*tile, 3)
    x = torch.rand((ci, H, W), generator=g, device="cuda")
    w = torch.randn((co, ci, k, k), generator=g, device="cuda") * (2.0 / (ci * k * k)) ** 0.5
    y, ref = full_update(x, w).double(), conv64(x, w)
    assert ((y - ref).norm() / ref.norm()).item() < 2.0 ** -24 * (1.5 * (ci * k * k / 32 / 6) ** 0.5 + 1)
