"""Attention at every head size the library takes and at the edges of its 32-row blocks: sequences of 1, 31, 32, 33 and a
few blocks more, all masks, against the oracle in 64 bits; and what a position that nobody may see holds must not show."""
import math

import numpy as np
import pytest
import torch

from oracle import block as ob
from paper_2006_09503_amd import binding as B
from paper_2006_09503_amd.synth import round_to_bf16

from gpu_util import rel, to_dev, to_host

pytestmark = pytest.mark.gpu

F32, BF16 = 0, 1
# fp32: sums of up to 128 (scores) and 200 (rows) products, each rounded to 2^-24: about sqrt(200) * 6e-8 per operand pass.
# bf16: one rounding of the result (2^-9 / sqrt(3) = 1.1e-3 rms) plus, in the gradient, that of O inside delta.
TOL = {F32: 4e-6, BF16: 3.5e-3}


def run_attention(dtype, b, s, a, dh, mask, qkv, d_o, lens):
    h = a * dh
    L = B.lib()
    QKV, DO = to_dev(qkv, dtype), to_dev(d_o, dtype)
    LEN = None if lens is None else torch.from_numpy(lens).cuda()
    lp = None if LEN is None else LEN.data_ptr()
    dt = torch.bfloat16 if dtype == BF16 else torch.float32
    O = torch.full((b, s, h), float("nan"), device="cuda", dtype=dt)
    D = torch.full((b, s, 3 * h), float("nan"), device="cuda", dtype=dt)
    lse = torch.empty((b, a, s), device="cuda")
    delta = torch.empty((b, a, s), device="cuda")
    assert L.k2bw_attention_fwd(dtype, b, s, a, dh, mask, lp, QKV.data_ptr(), O.data_ptr(), lse.data_ptr(), None) == 0
    assert L.k2bw_attention_bwd(dtype, b, s, a, dh, mask, lp, QKV.data_ptr(), O.data_ptr(), lse.data_ptr(), DO.data_ptr(), D.data_ptr(),
                                delta.data_ptr(), None, 0, None, None) == 0
    torch.cuda.synchronize()
    return to_host(O), to_host(lse), to_host(D)


def draw(dtype, b, s, a, dh, mask):
    rng = np.random.default_rng(b * 1000 + s * 7 + a + dh * 13 + mask)
    q = lambda z: round_to_bf16(z) if dtype == BF16 else z
    qkv = q(rng.standard_normal((b, s, 3 * a * dh)).astype(np.float32))
    d_o = q(rng.standard_normal((b, s, a * dh)).astype(np.float32))
    lens = rng.integers(1, s + 1, size=b).astype(np.int32) if mask == 2 else None
    return qkv, d_o, lens


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("dh", [8, 16, 40, 48, 56, 72, 88, 96, 104, 112, 120, 128])
@pytest.mark.parametrize("b,s,a,mask", [(2, 1, 2, 2), (1, 31, 3, 1), (2, 33, 1, 0), (1, 32, 1, 1), (2, 200, 2, 2), (1, 300, 1, 1)])
def test_attention_at_every_head_size(dtype, dh, b, s, a, mask):
    h = a * dh
    qkv, d_o, lens = draw(dtype, b, s, a, dh, mask)
    O, lse, D = run_attention(dtype, b, s, a, dh, mask, qkv, d_o, lens)
    split = lambda z: z.reshape(s, a, dh).transpose(1, 0, 2).astype(np.float64)
    back = lambda z: z.transpose(1, 0, 2).reshape(s, h)
    tol = TOL[dtype] if dtype == F32 or dh not in (32, 64, 80, 128) else 6e-3   # (those four keep bf16 probabilities)
    for n in range(b):
        q, k, v = (split(qkv[n, :, i * h:(i + 1) * h]) for i in range(3))
        vis = ob.visibility(mask, s, None if lens is None else int(lens[n]))
        o, P = ob.attention_fwd(q, k, v, vis)
        dq, dk, dv = ob.attention_bwd(split(d_o[n]), q, k, v, P)
        S = np.where(vis[None], q @ k.transpose(0, 2, 1) / math.sqrt(dh), -np.inf)
        want_lse = np.log(np.exp(S - S.max(-1, keepdims=True)).sum(-1)) + S.max(-1)
        assert rel(O[n], back(o)) < tol
        assert np.abs(lse[n] - want_lse).max() < (1e-5 if dtype == F32 else 1e-4)
        # (a row that sees one key has exactly zero dQ and dK: compare against the size of the whole gradient)
        size = max(np.linalg.norm(g) for g in (dq, dk, dv))
        for i, g in enumerate((dq, dk, dv)):
            assert np.linalg.norm(D[n, :, i * h:(i + 1) * h] - back(g)) < 2 * tol * size
        if mask == 2:
            assert np.all(D[n, lens[n]:, h:] == 0.0)


@pytest.mark.parametrize("dtype,dh", [(F32, 32), (F32, 72), (F32, 128), (BF16, 96), (BF16, 40)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_what_nobody_sees_does_not_show(dtype, dh, bad):
    """Causal: a non-finite key or value at position 40 leaves the results of queries 0..39 as they are, and a non-finite
    output gradient of query 40 the gradients of keys 41..69 (up to the order of a sum, which a tile with such values takes
    row by row).  Padding: keys past the length may hold anything."""
    same = lambda x, y: rel(y, x.astype(np.float64)) < (2e-6 if dtype == F32 else 3e-3)
    b, s, a = 1, 70, 2
    h = a * dh
    qkv, d_o, _ = draw(dtype, b, s, a, dh, 1)
    O0, lse0, D0 = run_attention(dtype, b, s, a, dh, 1, qkv, d_o, None)
    poisoned = qkv.copy()
    poisoned[0, 40, h:] = bad                       # K and V of one token
    O1, lse1, D1 = run_attention(dtype, b, s, a, dh, 1, poisoned, d_o, None)
    assert same(O0[0, :40], O1[0, :40]) and same(lse0[0, :, :40], lse1[0, :, :40])
    assert same(D0[0, :40, :h], D1[0, :40, :h])                  # dQ of queries that do not see it
    g = d_o.copy()
    g[0, 40] = bad                                  # the gradient of one query
    O2, lse2, D2 = run_attention(dtype, b, s, a, dh, 1, qkv, g, None)
    assert same(D0[0, 41:, h:], D2[0, 41:, h:])                  # dK, dV of the keys it does not see
    lens = np.array([50], dtype=np.int32)
    O3, lse3, D3 = run_attention(dtype, b, s, a, dh, 2, qkv, d_o, lens)
    poisoned = qkv.copy()
    poisoned[0, 50:, h:] = bad
    O4, lse4, D4 = run_attention(dtype, b, s, a, dh, 2, poisoned, d_o, lens)
    assert np.array_equal(O3, O4) and np.array_equal(lse3, lse4) and np.array_equal(D3, D4)


@pytest.mark.parametrize("dh", [24, 40, 56, 72, 96, 112, 120])
@pytest.mark.parametrize("b,a", [(1, 2), (4, 16), (9, 16)])
def test_probabilities_keep_their_32_bits(dh, b, a):
    """bf16 at the head sizes without bf16 probabilities: P and dS enter the second products with all their bits.  Rows of
    +-1 or +-1024 in turn against nearly equal P or dS: what remains of each sum is some 1e-3 of its terms, so 16 bits of P or dS
    would show as 2^-17 * 1e3 = 8e-3, while rounding the result to bf16 is at most 2^-9 and 32-bit terms leave 2^-24 * 1e3."""
    s, h = 256, a * dh
    rng = np.random.default_rng(dh + b)
    alt = np.where(np.arange(s) % 2 == 0, 1024.0, -1024.0)
    q, k, v, g = (rng.standard_normal((b, a, s, dh)) for _ in range(4))
    q *= 4e-4
    q[..., 0] = 0.0                                  # column 0 of the keys does not enter the scores
    k[..., 0] = alt
    v[..., 1::2, :] = v[..., 0::2, :]                # neighbours share dP but for column 0,
    v[..., 0] = alt / 1024
    g[..., 0] *= 4e-4                                # which adds as little as P differs by
    g[..., 1] = alt / 1024
    q, k, v, g = (round_to_bf16(t.astype(np.float32)).astype(np.float64) for t in (q, k, v, g))
    join = lambda t: t.transpose(0, 2, 1, 3).reshape(b, s, h).astype(np.float32)
    O, lse, D = run_attention(BF16, b, s, a, dh, 0, np.concatenate([join(q), join(k), join(v)], -1), join(g), None)
    split = lambda t: t.reshape(b, s, a, dh).transpose(0, 2, 1, 3).astype(np.float64)
    S = q @ k.transpose(0, 1, 3, 2) / math.sqrt(dh)
    P = np.exp(S - S.max(-1, keepdims=True))
    P /= P.sum(-1, keepdims=True)
    dS = P * (g @ v.transpose(0, 1, 3, 2) - (g * split(O)).sum(-1, keepdims=True))
    tol = 2.0 ** -9 + 6e-4
    assert rel(split(O)[..., 0], (P @ v)[..., 0]) < tol
    assert rel(split(D[..., 2 * h:])[..., 1], (P.transpose(0, 1, 3, 2) @ g)[..., 1]) < tol
    assert rel(split(D[..., :h])[..., 0], (dS @ k)[..., 0] / math.sqrt(dh)) < tol


@pytest.mark.parametrize("dtype,dh", [(F32, 32), (F32, 72), (BF16, 64), (BF16, 40)])
@pytest.mark.parametrize("s,key", [(33, 32), (33, 0), (200, 130)])
def test_a_visible_nan_reaches_the_log_sum(dtype, dh, s, key):
    """A NaN in a visible key makes o and lse of every row NaN, also where it is the only key of its tile (s = 33, key 32) and the
    waves that share the keys see nothing but it; a NaN in a query makes that row's NaN and leaves the others alone."""
    h = 2 * dh
    qkv, d_o, _ = draw(dtype, 1, s, 2, dh, 0)
    O0, lse0, _ = run_attention(dtype, 1, s, 2, dh, 0, qkv, d_o, None)
    bad = qkv.copy()
    bad[0, key, h:2 * h] = float("nan")
    O, lse, _ = run_attention(dtype, 1, s, 2, dh, 0, bad, d_o, None)
    assert np.isnan(O).all() and np.isnan(lse).all()
    bad = qkv.copy()
    bad[0, 5, :h] = float("nan")
    O, lse, _ = run_attention(dtype, 1, s, 2, dh, 0, bad, d_o, None)
    others = np.arange(s) != 5
    assert np.isnan(O[0, 5]).all() and np.isnan(lse[0, :, 5]).all()
    assert np.array_equal(O[0, others], O0[0, others]) and np.array_equal(lse[0][:, others], lse0[0][:, others])


@pytest.mark.parametrize("dh", [32, 64, 80, 96, 128])
@pytest.mark.parametrize("b,s,a,mask", [(1, 200, 2, 1), (1, 330, 2, 0), (3, 300, 16, 0), (3, 330, 16, 2), (5, 300, 16, 1), (5, 270, 16, 0)])
def test_attention_at_every_split_of_the_streamed_rows(dh, b, s, a, mask):
    """Few, some and many workgroups: blocks of 64 and 128 rows whose two halves of waves take every second tile of the other
    side (odd and even numbers of tiles, halves that see nothing), and blocks of 256 rows that take all; with the bias gradient."""
    h = a * dh
    qkv, d_o, lens = draw(BF16, b, s, a, dh, mask)
    if lens is not None:
        lens[:2] = 1, 65
    L = B.lib()
    fused = dh != 96
    QKV, DO = to_dev(qkv, BF16), to_dev(d_o, BF16)
    lp = None if lens is None else (LEN := torch.from_numpy(lens).cuda()).data_ptr()
    n_ws = L.k2bw_attention_bwd_workspace(b, s, a, dh)
    ws = torch.full((n_ws + 64,), 7.0, device="cuda")
    db = torch.ones(3 * h, device="cuda")
    O = torch.full((b, s, h), float("nan"), device="cuda", dtype=torch.bfloat16)
    D = torch.full((b, s, 3 * h), float("nan"), device="cuda", dtype=torch.bfloat16)
    lse, delta = torch.empty((b, a, s), device="cuda"), torch.empty((b, a, s), device="cuda")
    assert L.k2bw_attention_fwd(BF16, b, s, a, dh, mask, lp, QKV.data_ptr(), O.data_ptr(), lse.data_ptr(), None) == 0
    assert L.k2bw_attention_bwd(BF16, b, s, a, dh, mask, lp, QKV.data_ptr(), O.data_ptr(), lse.data_ptr(), DO.data_ptr(), D.data_ptr(),
                                delta.data_ptr(), db.data_ptr() if fused else None, 1, ws.data_ptr() if fused else None, None) == 0
    torch.cuda.synchronize()
    assert bool((ws[n_ws:] == 7.0).all())
    split = lambda z: z.reshape(s, a, dh).transpose(1, 0, 2).astype(np.float64)
    back = lambda z: z.transpose(1, 0, 2).reshape(s, h)
    tol = 6e-3 if fused else TOL[BF16]
    got_o, got_lse, got_d = to_host(O), to_host(lse), to_host(D)
    for n in range(b):
        q, k, v = (split(qkv[n, :, i * h:(i + 1) * h]) for i in range(3))
        vis = ob.visibility(mask, s, None if lens is None else int(lens[n]))
        o, P = ob.attention_fwd(q, k, v, vis)
        grads = ob.attention_bwd(split(d_o[n]), q, k, v, P)
        S = np.where(vis[None], q @ k.transpose(0, 2, 1) / math.sqrt(dh), -np.inf)
        assert rel(got_o[n], back(o)) < tol
        assert np.abs(got_lse[n] - np.log(np.exp(S - S.max(-1, keepdims=True)).sum(-1)) - S.max(-1)).max() < 1e-4
        size = max(np.linalg.norm(g) for g in grads)
        for i, g in enumerate(grads):
            assert np.linalg.norm(got_d[n, :, i * h:(i + 1) * h] - back(g)) < 2 * tol * size
    if fused:   # b*s values, each within 2^-8 of its own rounded one: their rounding errors add up like sqrt
        want = got_d.astype(np.float64).reshape(-1, 3 * h)
        bound = 2.0 ** -9 * np.sqrt((want ** 2).sum(0)) * 4 + 1e-5 * np.abs(want).sum(0) + 1e-6
        assert np.all(np.abs(to_host(db) - 1.0 - want.sum(0)) < bound)
