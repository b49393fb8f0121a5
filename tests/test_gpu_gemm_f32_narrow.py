"""fp32 products of at most one 16 x 16 tile per CU: edges of the tiles, every remainder of the chunks of 16 k (and of the loads of 4), one wave's
chunk, all waves' chunks and more than the waves hold at once, both sides of the rule on the number of tiles.  (No single element: a GELU of -3
is 1 + erf = 1e-3, of which fp32 leaves 6e-8 / 1e-3, more than the bound on the norm of a whole matrix.)"""
import pytest

from test_gpu_gemm_small import test_fp32_products_at_tile_edges as products

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 40, 4), (16, 16, 16), (15, 17, 20), (17, 15, 124), (33, 47, 128), (16, 48, 132), (31, 80, 256), (48, 33, 260),
                                   (20, 36, 1024), (65, 19, 1036), (9, 100, 2052), (256, 256, 64), (257, 256, 64), (240, 272, 520), (40, 40, 18)])
@pytest.mark.parametrize("pad", [0, 4, 1])
def test_products_of_16x16_tiles(M, N, K, pad):
    for tb in (0, 1):
        products(M, N, K, 0, tb, pad)


@pytest.mark.parametrize("M,N,K", [(16, 4096, 300), (1, 4088, 272), (15, 672, 288), (570, 20, 320), (33, 1350, 508), (4096, 12, 260)])
def test_flat_products_and_reductions_just_above_two_chunks_per_wave(M, N, K):
    """One row or column of tiles, up to one tile per CU; waves with two and with three chunks."""
    for tb in (0, 1):
        products(M, N, K, 0, tb, 4)
