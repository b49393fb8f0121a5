"""The phased bf16 GEMM kernels, forced, where they can go wrong: one K tile, an odd and an even number of them, a partial one in front;
matrices smaller than a tile, tiles cut by the edge in either part of their rows; launches that end in tiles of half the height; a
segmented reduction range.  NaNs lie behind every row and every matrix."""
import pytest

from paper_2006_09503_amd import binding as B
from test_gpu_gemm_small import test_bf16_partial_k_tiles as partial_k_tiles
from test_gpu_gemm_small import test_bf16_weight_gradient_of_any_number_of_tokens as any_number_of_tokens
from test_gpu_kernels import test_gemm_every_tile_variant as every_form
from test_gpu_kernels import test_gemm_weight_gradient_over_several_microbatches as several_microbatches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [25, 26, 27])
@pytest.mark.parametrize("M,N,K", [(8, 8, 64), (72, 264, 72), (136, 520, 128), (264, 248, 136), (160, 256, 192), (328, 272, 1016), (456, 512, 320)])
def test_forward_and_data_gradient(tile, M, N, K):
    partial_k_tiles(tile, M, N, K)


@pytest.mark.parametrize("M,N,K", [(8, 8, 64), (72, 264, 65), (136, 520, 127), (264, 248, 128), (160, 256, 200), (328, 272, 1000)])
def test_weight_gradient(M, N, K):
    any_number_of_tokens(27, M, N, K)


@pytest.mark.parametrize("M,N,K", [(4360, 4096, 64), (4096, 4360, 136)])
def test_tiles_of_half_the_height_end_a_launch(M, N, K):
    """18 x 16 and 16 x 18 tiles of 256 x 256: the last rows of tiles run as tiles of 128 rows.  (Their partial sums of the fused bias
    gradient: test_gemm_gelu_gradient_with_fused_bias_gradient.)"""
    every_form(25, M, N, K)


@pytest.mark.parametrize("M,N,T,idx_a,idx_b", [(520, 264, 64, [3, 0, 2], [0, 1, 2]), (136, 520, 192, [1, 4], [2, 0])])   # (pieces of whole K tiles)
def test_weight_gradient_over_pieces_in_several_buffers(M, N, T, idx_a, idx_b):
    L = B.lib()
    assert L.k2bw_tune_gemm_tile(27) == 0
    try:
        several_microbatches(M, N, T, idx_a, idx_b)
    finally:
        assert L.k2bw_tune_gemm_tile(0) == 0
