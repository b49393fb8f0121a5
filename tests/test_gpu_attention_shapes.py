"""Every shape of an attention launch (rows per workgroup, streamed rows split or not, waves) at ragged sizes, with the shape that ran
read back from what the backward pass leaves in its workspace, against the same in 64 bits."""
import math

import pytest
import torch

from paper_2006_09503_amd import binding as B

pytestmark = pytest.mark.gpu

F32, BF16 = 0, 1
FUSED = (32, 64, 80, 128)            # bf16 head sizes whose backward also returns the bias gradient, with bf16 probabilities
TOL = {F32: 4e-6, BF16: 3.5e-3}      # see test_gpu_attention_heads.py; 6e-3 with bf16 probabilities


def reference(qkv, d_o, a, mask, lens):
    """(o, lse, dqkv) in 64 bits."""
    b, s, h3 = qkv.shape
    dh = h3 // 3 // a
    q, k, v = (t.reshape(b, s, a, dh).transpose(1, 2).reshape(b * a, s, dh).contiguous() for t in qkv.double().split(h3 // 3, -1))
    g = d_o.double().reshape(b, s, a, dh).transpose(1, 2).reshape(b * a, s, dh).contiguous()
    i = torch.arange(s, device="cuda")
    if mask == 1:
        vis = (i[None, :] <= i[:, None])[None]
    elif mask == 2:
        vis = (i[None, :] < lens[:, None]).repeat_interleave(a, 0)[:, None, :].expand(b * a, s, s)
    else:
        vis = torch.ones((1, s, s), dtype=torch.bool, device="cuda")
    S = (torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(dh)).masked_fill(~vis, -math.inf)
    P = torch.softmax(S, -1)
    o = torch.bmm(P, v)
    dS = P * (torch.bmm(g, v.transpose(1, 2).contiguous()) - (g * o).sum(-1, keepdim=True))
    grads = (torch.bmm(dS, k) / math.sqrt(dh), torch.bmm(dS.transpose(1, 2).contiguous(), q) / math.sqrt(dh),
             torch.bmm(P.transpose(1, 2).contiguous(), g))
    back = lambda t: t.reshape(b, a, s, dh).transpose(1, 2).reshape(b, s, a * dh)
    return back(o), torch.logsumexp(S, -1).reshape(b, a, s), torch.cat([back(t) for t in grads], -1)


def run(dtype, b, s, a, dh, mask, qkv, d_o, lens, dbias=None, ws=None):
    L = B.lib()
    p = lambda t: None if t is None else t.data_ptr()
    o, dqkv = torch.full_like(d_o, math.nan), torch.full_like(qkv, math.nan)
    lse, delta = torch.empty((b, a, s), device="cuda"), torch.empty((b, a, s), device="cuda")
    assert L.k2bw_attention_fwd(dtype, b, s, a, dh, mask, p(lens), p(qkv), p(o), p(lse), None) == 0
    assert L.k2bw_attention_bwd(dtype, b, s, a, dh, mask, p(lens), p(qkv), p(o), p(lse), p(d_o), p(dqkv), p(delta), p(dbias), 1, p(ws),
                                None) == 0
    torch.cuda.synchronize()
    return o, lse, dqkv


def inputs(dtype, b, s, a, dh, mask):
    gen = torch.Generator(device="cuda").manual_seed(b * 1000 + s * 7 + a + dh * 13 + mask)
    dt = torch.bfloat16 if dtype == BF16 else torch.float32
    qkv = torch.randn((b, s, 3 * a * dh), generator=gen, device="cuda").to(dt)
    d_o = torch.randn((b, s, a * dh), generator=gen, device="cuda").to(dt)
    lens = None
    if mask == 2:
        lens = torch.randint(1, s + 1, (b,), generator=gen, device="cuda", dtype=torch.int32)
        lens[0], lens[1] = 1, min(s, 257)
    return qkv, d_o, lens


def blocks_per_head(b, s, a, mask):
    """How many workgroups the backward pass splits a head's rows into at the head sizes other than 128: the partial rows that head
    size 64 leaves."""
    qkv, d_o, lens = inputs(BF16, b, s, a, 64, mask)
    ws = torch.full((B.lib().k2bw_attention_bwd_workspace(b, s, a, 64),), math.nan, device="cuda")
    run(BF16, b, s, a, 64, mask, qkv, d_o, lens, torch.zeros(3 * a * 64, device="cuda"), ws)
    return int((~torch.isnan(ws)).sum()) // (3 * a * 64) // b


# (b, s, a, mask) and, with 256 CUs, the rows of a workgroup of the backward pass (head size 128: the second number)
SHAPES = [
    ((2, 300, 16, 0), 64, 64), ((2, 300, 16, 1), 64, 64), ((2, 300, 16, 2), 64, 64), ((2, 500, 16, 2), 64, 64),   # dK and dV together
    ((20, 60, 8, 0), 64, 256), ((40, 60, 8, 2), 64, 256),                                                        # one tile
    ((3, 330, 16, 2), 128, 128), ((5, 300, 16, 1), 128, 128), ((6, 330, 16, 1), 128, 256),
    ((9, 270, 16, 1), 256, 256), ((5, 300, 16, 2), 256, 256), ((5, 270, 16, 0), 256, 256), ((16, 131, 16, 1), 256, 256),
    ((8, 330, 16, 1), 256, 256),
]


@pytest.mark.parametrize("dh", [24, 32, 40, 56, 64, 72, 80, 96, 112, 120, 128])
@pytest.mark.parametrize("shape,rows,rows128", SHAPES)
def test_every_launch_shape_at_ragged_sizes(shape, rows, rows128, dh):
    b, s, a, mask = shape
    h = a * dh
    fused = dh in FUSED
    qkv, d_o, lens = inputs(BF16, b, s, a, dh, mask)
    n_ws = B.lib().k2bw_attention_bwd_workspace(b, s, a, dh)
    ws = torch.full((n_ws + 64,), math.nan, device="cuda") if fused else None
    db = torch.ones(3 * h, device="cuda") if fused else None
    o, lse, dqkv = run(BF16, b, s, a, dh, mask, qkv, d_o, lens, db, ws)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:   # the rule counts CUs
        want = rows128 if dh == 128 else rows
        if fused:
            assert int((~torch.isnan(ws)).sum()) == b * -(-s // want) * 3 * h
        else:
            assert blocks_per_head(b, s, a, mask) == -(-s // want)
    o64, lse64, d64 = reference(qkv, d_o, a, mask, lens)
    tol = 6e-3 if fused else TOL[BF16]
    rel = lambda x, y: float((x.double() - y).norm() / y.norm())
    assert rel(o, o64) < tol
    assert float((lse.double() - lse64).abs().max()) < 1e-4
    size = max(float(t.norm()) for t in d64.split(h, -1))
    for got, want in zip(dqkv.split(h, -1), d64.split(h, -1)):
        assert float((got.double() - want).norm()) < 2 * tol * size
    if mask == 2:
        for n in range(b):
            assert bool((dqkv[n, int(lens[n]):, h:] == 0).all())
    if fused:   # b*s values, each within 2^-8 of its own rounded one: their rounding errors add up like sqrt
        d = dqkv.double().reshape(-1, 3 * h)
        bound = 2.0 ** -9 * 4 * (d ** 2).sum(0).sqrt() + 1e-5 * d.abs().sum(0) + 1e-6
        assert bool(((db.double() - 1.0 - d.sum(0)).abs() < bound).all())


@pytest.mark.parametrize("dh", [40, 96, 112])
@pytest.mark.parametrize("shape,rows,pos", [((2, 300, 16), 64, 200), ((5, 300, 16), 128, 200), ((9, 270, 16), 256, 260)])
@pytest.mark.parametrize("bad", [math.nan, math.inf])
def test_what_nobody_sees_does_not_show_in_any_launch_shape(shape, rows, pos, dh, bad):
    """The restart of a workgroup that meets an infinity or a NaN in a tile that some of its rows may not see, in blocks that are
    not the first: causal, the key and value of token `pos` in one head's columns, then the gradient of that query."""
    b, s, a = shape
    h = a * dh
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert blocks_per_head(b, s, a, 1) == -(-s // rows)
    qkv, d_o, _ = inputs(BF16, b, s, a, dh, 1)
    o0, lse0, d0 = run(BF16, b, s, a, dh, 1, qkv, d_o, None)
    same = lambda x, y: float((x.double() - y.double()).norm() / y.double().norm()) < 3e-3   # (the order of a sum, then bf16)
    poisoned = qkv.clone()
    poisoned[:, pos, h:] = bad
    o1, lse1, d1 = run(BF16, b, s, a, dh, 1, poisoned, d_o, None)
    assert same(o1[:, :pos], o0[:, :pos]) and same(lse1[:, :, :pos], lse0[:, :, :pos]) and same(d1[:, :pos, :h], d0[:, :pos, :h])
    assert bool(torch.isnan(o1[:, pos:]).all())     # and it shows where it is seen
    poisoned = d_o.clone()
    poisoned[:, pos] = bad
    _, _, d2 = run(BF16, b, s, a, dh, 1, qkv, poisoned, None)
    assert same(d2[:, pos + 1:, h:], d0[:, pos + 1:, h:])
    lens = torch.full((b,), pos, device="cuda", dtype=torch.int32)
    o3, lse3, d3 = run(BF16, b, s, a, dh, 2, qkv, d_o, lens)
    poisoned = qkv.clone()
    poisoned[:, pos:, h:] = bad
    o4, lse4, d4 = run(BF16, b, s, a, dh, 2, poisoned, d_o, lens)
    assert torch.equal(o3, o4) and torch.equal(lse3, lse4) and torch.equal(d3, d4)


@pytest.mark.parametrize("dh", [8, 40, 64, 72, 96, 112, 128])
@pytest.mark.parametrize("b,s,a,mask", [(40, 31, 8, 1), (33, 1, 8, 2), (40, 32, 8, 0), (40, 29, 7, 2), (40, 33, 8, 1),
                                        (30, 100, 8, 2), (30, 97, 8, 1), (20, 70, 8, 1), (8, 40, 8, 2)])
def test_fp32_launches_of_many_blocks_on_one_wave(dh, b, s, a, mask):
    """Enough blocks of 32 rows for every SIMD, one to four tiles each (too few, four waves: the last, and the two before it in the
    backward pass of heads up to 64)."""
    h = a * dh
    qkv, d_o, lens = inputs(F32, b, s, a, dh, mask)
    o, lse, dqkv = run(F32, b, s, a, dh, mask, qkv, d_o, lens)
    o64, lse64, d64 = reference(qkv, d_o, a, mask, lens)
    assert float((o.double() - o64).norm() / o64.norm()) < TOL[F32]
    assert float((lse.double() - lse64).abs().max()) < 1e-5
    size = max(float(t.norm()) for t in d64.split(h, -1))
    for got, want in zip(dqkv.split(h, -1), d64.split(h, -1)):
        assert float((got.double() - want).norm()) < 2 * TOL[F32] * size
