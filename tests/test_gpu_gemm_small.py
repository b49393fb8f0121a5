"""Products at the edges of their kernels' tiles.

fp32: at the edges of the tiles and of the split reduction range: one row, one column, 31/32/33, 63/64/65, reduction
ranges from 1 to a few chunks of 16 with every kind of remainder, leading dimensions that allow no 16-byte loads; all forms and
epilogues, and several products in one launch through the weight-gradient accumulation of a stage.
bf16: partial K tiles of the direct-to-LDS kernels (every remainder class of their K tiles, with NaNs behind the matrices, which
must not show), and the kernels that split the reduction range over a workgroup's waves."""
import numpy as np
import pytest
import torch

from oracle import block as ob
from paper_2006_09503_amd import binding as B

from paper_2006_09503_amd.synth import round_to_bf16

from gpu_util import gemm_tile_cases, gemm_tile_runs, rel, to_host

pytestmark = pytest.mark.gpu

# the last two pick 32 x 32 tiles in several rounds, and 128 x 128 tiles, by the rule on sizes
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


@pytest.mark.parametrize("M,N,K", [(930, 1030, 601), (1450, 2600, 9), (2049, 1290, 40), (130, 4100, 200)])
def test_fp32_products_on_both_sides_of_the_tile_rule(M, N, K):
    """64 x 64 tiles (one round, long reduction), and wide outputs whose short reductions stay on 128 x 128 tiles."""
    for ta, tb in ((0, 0), (0, 1), (1, 0), (1, 1)):
        test_fp32_products_at_tile_edges(M, N, K, ta, tb, 0)


BF16 = 1


def bf16_matrix(rng, rows, cols, ld, scale=1.0):
    """A bf16 matrix with rows `ld` apart and NaN everywhere else, a row's worth behind the end included."""
    a = round_to_bf16((rng.standard_normal((rows, cols)) * scale).astype(np.float32))
    d = torch.full((rows + 1, ld), float("nan"), device="cuda", dtype=torch.bfloat16)
    d[:rows, :cols] = torch.from_numpy(a).cuda().to(torch.bfloat16)
    return a.astype(np.float64), d


@pytest.mark.parametrize("tile,M,N,K", gemm_tile_cases([0, 2, 22, 23, 24, 32, 64], [(8, 8, 8), (40, 72, 40), (264, 136, 72), (136, 264, 104),
                                                                                 (96, 520, 200), (328, 272, 1016), (72, 64, 2056)], "fd"))
def test_bf16_partial_k_tiles(tile, M, N, K):
    """Forward and data gradient in the forms that have the tile."""
    rng = np.random.default_rng(M + N + K + tile)
    L = B.lib()
    assert L.k2bw_tune_gemm_tile(tile) == 0
    try:
        x, X = bf16_matrix(rng, M, K, K + 8)
        w, W = bf16_matrix(rng, K, N, N + 8, 0.1)
        wt, Wt = bf16_matrix(rng, N, K, K + 8, 0.1)
        bias, Bi = bf16_matrix(rng, 1, N, N)
        aux, U = bf16_matrix(rng, M, N, N)
        C = torch.empty((M, N), device="cuda", dtype=torch.bfloat16)
        G = torch.empty_like(C)
        for tb, (m, dev, ld) in ((0, (w, W, N + 8)), (1, (wt.T, Wt, K + 8))):
            if not gemm_tile_runs(tile, "fd"[tb], K):
                continue
            want = x @ m
            for epi in (0, 1, 2):
                if tb and epi == 1:
                    continue   # a form nobody issues
                assert L.k2bw_gemm(BF16, 0, tb, epi, M, N, K, X.data_ptr(), K + 8, dev.data_ptr(), ld, C.data_ptr(), N,
                                   Bi.data_ptr() if epi < 2 else None, U.data_ptr() if epi != 1 else None,
                                   G.data_ptr() if epi == 1 else None, 0, None) == 0
                torch.cuda.synchronize()
                full = {0: want + bias + aux, 1: want + bias, 2: want * ob.gelu_grad(aux)}[epi]
                assert rel(to_host(C), full) < 3e-3      # one rounding to bf16: 2^-9 / sqrt(3), and the fast GELU
                if epi == 1:
                    assert rel(to_host(G), ob.gelu(full)) < 3e-3
        if not gemm_tile_runs(tile, "d", K):
            return
        # the fused bias gradient: column sums of the unrounded values
        db = torch.full((N,), float("nan"), device="cuda")
        ws = torch.empty(L.k2bw_gemm_dgrad_gelu_bias_workspace(M, N), device="cuda")
        assert L.k2bw_gemm_dgrad_gelu_bias(M, N, K, X.data_ptr(), K + 8, Wt.data_ptr(), K + 8, C.data_ptr(), N, U.data_ptr(), db.data_ptr(),
                                           0, ws.data_ptr(), None) == 0
        torch.cuda.synchronize()
        full = (x @ wt.T) * ob.gelu_grad(aux)
        assert np.abs(to_host(db) - full.sum(0)).max() < 1e-4 * np.sqrt((full ** 2).sum(0)).max() * np.sqrt(M)
    finally:
        assert L.k2bw_tune_gemm_tile(0) == 0


@pytest.mark.parametrize("tile,M,N,K", gemm_tile_cases([0, 2, 22, 23, 24, 32, 64], [(72, 40, 1), (136, 264, 33), (264, 136, 65), (256, 520, 127),
                                                                                 (520, 264, 1000), (64, 64, 4099)], "w"))
def test_bf16_weight_gradient_of_any_number_of_tokens(tile, M, N, K):
    assert gemm_tile_runs(tile, "w", K)
    rng = np.random.default_rng(M + N + K + tile)
    L = B.lib()
    assert L.k2bw_tune_gemm_tile(tile) == 0
    try:
        x, X = bf16_matrix(rng, K, M, M + 8)
        dy, D = bf16_matrix(rng, K, N, N + 8)
        g0 = rng.standard_normal((M, N)).astype(np.float32)
        for acc in (0, 1):
            G = torch.from_numpy(g0.copy()).cuda()
            assert L.k2bw_gemm(BF16, 1, 0, 3, M, N, K, X.data_ptr(), M + 8, D.data_ptr(), N + 8, G.data_ptr(), N, None, None, None, acc,
                               None) == 0
            torch.cuda.synchronize()
            assert rel(to_host(G), x.T @ dy + (g0 if acc else 0)) < 2e-6
    finally:
        assert L.k2bw_tune_gemm_tile(0) == 0


@pytest.mark.parametrize("M,N,K", [(200, 17000, 72), (1168, 3304, 1544), (648, 11960, 40), (4104, 2056, 96), (968, 5944, 520), (392, 8536, 1032),
                                   (1000, 2312, 2104), (3080, 3592, 40), (136, 10296, 264), (1304, 4736, 56), (1592, 8976, 96), (1752, 1320, 48)])
def test_bf16_products_on_both_sides_of_the_tile_rule(M, N, K):
    """The tile the library picks, around its lines: 128 x 128 tiles in several rounds of short and long reductions, 192 x 256 and
    256 x 256 tiles, reductions that are whole 128-byte lines and that are not, or less than one; the partial K tiles and NaNs of the tests above."""
    for k in (K, K + (-K) % 64):
        test_bf16_partial_k_tiles(0, M, N, k)
        test_bf16_weight_gradient_of_any_number_of_tokens(0, M, N, k - 3)


@pytest.mark.parametrize("dtype", [0, BF16])
@pytest.mark.parametrize("rows,n", [(1, 8), (127, 40), (129, 24), (513, 264), (1024, 72), (1025, 4104), (2048, 4096), (2049, 32),
                                    (256, 32768), (257, 28672), (511, 14336), (520, 13912), (1024, 8200), (1500, 2504)])
def test_column_sums_on_both_sides_of_the_one_launch_rule(dtype, rows, n):
    rng = np.random.default_rng(rows + n)
    y = rng.standard_normal((rows, n)).astype(np.float32)
    y = round_to_bf16(y) if dtype else y
    Y = torch.from_numpy(y).cuda().to(torch.bfloat16 if dtype else torch.float32)
    L = B.lib()
    ws = torch.empty(L.k2bw_bias_grad_workspace(n), device="cuda")
    out = torch.full((n,), float("nan"), device="cuda")
    for acc in (0, 1):
        assert L.k2bw_bias_grad(dtype, rows, n, Y.data_ptr(), out.data_ptr(), acc, ws.data_ptr(), None) == 0
    torch.cuda.synchronize()
    # sums of `rows` terms of size 1, each addition rounded to 2^-24 of a running sum of about sqrt(rows)
    assert np.abs(to_host(out) - 2 * y.astype(np.float64).sum(0)).max() < 1e-6 * rows + 1e-6


def test_column_sums_of_one_launch_round_no_more_than_a_tree():
    """128 rows, one to a thread: a tree of 7 additions per column, each off by 2^-24 / sqrt(3) of its result, leaves sqrt(7) of that;
    eight and then sixteen partial sums one after the other leave more."""
    L = B.lib()
    n, err, size = 3072, 0.0, 0.0
    ws = torch.empty(L.k2bw_bias_grad_workspace(n), device="cuda")
    out = torch.empty(n, device="cuda")
    for seed in range(6):
        y = torch.randn((128, n), device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed))
        assert L.k2bw_bias_grad(0, 128, n, y.data_ptr(), out.data_ptr(), 0, ws.data_ptr(), None) == 0
        torch.cuda.synchronize()
        want = y.double().sum(0)
        err += float(((out.double() - want) ** 2).sum())
        size += float((want ** 2).sum())
    assert (err / size) ** 0.5 < 7 ** 0.5 * 2.0 ** -24 / 3 ** 0.5
