"""fp32 products at the edges of the tiles and of the split reduction range: one row, one column, 31/32/33, 63/64/65, reduction
ranges from 1 to a few chunks of 16 with every kind of remainder, leading dimensions that allow no 16-byte loads; all forms and
epilogues, and several products in one launch through the weight-gradient accumulation of a stage."""
import numpy as np
import pytest
import torch

from oracle import block as ob
from paper_2006_09503_amd import binding as B

from gpu_util import rel, to_host

pytestmark = pytest.mark.gpu

# the last two pick 64 x 64 tiles, and 128 x 128 tiles, by the rule on sizes
SHAPES = [(1, 8, 1), (31, 33, 17), (32, 32, 16), (33, 65, 31), (64, 63, 128), (65, 128, 130), (129, 40, 7), (1024, 1030, 40), (4100, 2052, 24)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("pad", [0, 4, 1])          # pad 1: rows that are not 16-byte aligned
def test_fp32_products_at_tile_edges(M, N, K, ta, tb, pad):
    rng = np.random.default_rng(M * 7 + N * 3 + K + ta + tb)
    L = B.lib()

    def matrix(rows, cols):
        a = rng.standard_normal((rows, cols)).astype(np.float32)
        d = torch.full((rows, cols + pad), float("nan"), device="cuda")   # what lies between the rows must not show
        d[:, :cols] = torch.from_numpy(a).cuda()
        return a.astype(np.float64), d, cols + pad

    a, A, lda = matrix(K, M) if ta else matrix(M, K)
    b, Bm, ldb = matrix(N, K) if tb else matrix(K, N)
    want = (a.T if ta else a) @ (b.T if tb else b)
    bias, BI, _ = matrix(1, N)
    aux, AU, ldc = matrix(M, N)
    tol = 3e-7 * np.sqrt(K) + 3e-7
    for epi, acc in ((0, 0), (1, 0), (2, 0), (3, 0), (3, 1)):
        C = torch.full((M, ldc), float("nan"), device="cuda")
        if acc:
            C[:, :N] = torch.from_numpy(aux.astype(np.float32)).cuda()
        G = torch.full((M, ldc), float("nan"), device="cuda")
        assert L.k2bw_gemm(0, ta, tb, epi, M, N, K, A.data_ptr(), lda, Bm.data_ptr(), ldb, C.data_ptr(), ldc,
                           BI.data_ptr() if epi < 2 else None, AU.data_ptr() if epi in (0, 2) else None,
                           G.data_ptr() if epi == 1 else None, acc, None) == 0
        torch.cuda.synchronize()
        c = to_host(C)[:, :N]
        full = {0: want + bias + aux, 1: want + bias, 2: want * ob.gelu_grad(aux), 3: want + (aux if acc else 0)}[epi]
        assert rel(c, full) < tol
        if epi == 1:
            assert rel(to_host(G)[:, :N], ob.gelu(full)) < tol
        assert bool(torch.isnan(C[:, N:]).all())
