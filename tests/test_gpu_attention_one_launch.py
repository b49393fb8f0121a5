"""bf16 attention, backward in one launch and in two: sizes on both sides of that rule in every launch shape (64, 128 and 256 rows per
workgroup), the longest sequence whose deltas a workgroup holds and one more, with the bias gradient where the kernels emit it; and
what a position that nobody may see holds must not show."""
import math

import pytest
import torch

from paper_2006_09503_amd import binding as B
from test_gpu_attention_shapes import BF16, FUSED, TOL, inputs, reference, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [32, 64, 80, 128, 16, 48, 72, 96, 112])
@pytest.mark.parametrize("b,s,a,mask", [(2, 65, 3, 1), (2, 500, 4, 0), (2, 500, 8, 2), (3, 500, 8, 1), (2, 1000, 8, 1), (16, 99, 8, 0), (30, 70, 12, 2),
                                        (30, 200, 12, 1), (2, 2048, 1, 2), (2, 2049, 1, 1)])
def test_backward_on_both_sides_of_the_launch_rule(dh, b, s, a, mask):
    h = a * dh
    qkv, d_o, lens = inputs(BF16, b, s, a, dh, mask)
    fused = dh in FUSED
    ws = torch.empty(B.lib().k2bw_attention_bwd_workspace(b, s, a, dh), device="cuda") if fused else None
    db = torch.ones(3 * h, device="cuda") if fused else None
    o, lse, dqkv = run(BF16, b, s, a, dh, mask, qkv, d_o, lens, db, ws)
    o64, lse64, d64 = reference(qkv, d_o, a, mask, lens)
    tol = 6e-3 if fused else TOL[BF16]
    assert float((o.double() - o64).norm() / o64.norm()) < tol
    assert float((lse.double() - lse64).abs().max()) < 1e-4
    size = max(float(t.norm()) for t in d64.split(h, -1))
    for got, want in zip(dqkv.split(h, -1), d64.split(h, -1)):
        assert float((got.double() - want).norm()) < 2 * tol * size
    if fused:   # sums of b * s values each off by tol of their rms, at random
        want = d64.sum((0, 1)) + 1
        assert float((db.double() - want).abs().max()) < 6 * tol * size / math.sqrt(3 * h)


@pytest.mark.parametrize("dh", [48, 96, 112])
@pytest.mark.parametrize("b,s,a,pos", [(1, 100, 2, 40), (2, 300, 8, 170), (20, 200, 12, 130)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_what_nobody_sees_does_not_show(dh, b, s, a, pos, bad):
    h = a * dh
    same = lambda x, y: bool(torch.isfinite(x).all()) and float((x.double() - y.double()).norm() / y.double().norm()) < 3e-3
    qkv, d_o, _ = inputs(BF16, b, s, a, dh, 1)
    _, _, d0 = run(BF16, b, s, a, dh, 1, qkv, d_o, None)
    poisoned = qkv.clone()
    poisoned[:, pos, h:] = bad                       # K and V of one token
    _, _, d1 = run(BF16, b, s, a, dh, 1, poisoned, d_o, None)
    assert same(d1[:, :pos, :h], d0[:, :pos, :h])
    poisoned = d_o.clone()
    poisoned[:, pos] = bad                           # the gradient of one query
    _, _, d2 = run(BF16, b, s, a, dh, 1, qkv, poisoned, None)
    assert same(d2[:, pos + 1:, h:], d0[:, pos + 1:, h:])


@pytest.mark.parametrize("dh", [32, 64, 96, 128])
@pytest.mark.parametrize("b,s,a,mask,one", [(2, 65, 3, 1, True), (1, 300, 4, 0, True), (2, 150, 2, 2, True), (2, 2049, 1, 1, False), (8, 900, 16, 0, False)])
def test_one_launch_hands_nothing_through_the_scratch_array(dh, b, s, a, mask, one):
    """Its workgroups run side by side, so what some of them left in delta others must not use: they get no pointer to it, and the caller's
    scratch array stays as it was.  In two launches it holds the row sums of dO * O afterwards."""
    h = a * dh
    qkv, d_o, lens = inputs(BF16, b, s, a, dh, mask)
    L, p = B.lib(), lambda t: None if t is None else t.data_ptr()
    o, dqkv = torch.empty_like(d_o), torch.empty_like(qkv)
    lse, delta = torch.empty((b, a, s), device="cuda"), torch.full((b, a, s), float("nan"), device="cuda")
    assert L.k2bw_attention_fwd(BF16, b, s, a, dh, mask, p(lens), p(qkv), p(o), p(lse), None) == 0
    assert L.k2bw_attention_bwd(BF16, b, s, a, dh, mask, p(lens), p(qkv), p(o), p(lse), p(d_o), p(dqkv), p(delta), None, 0, None, None) == 0
    torch.cuda.synchronize()
    assert bool(torch.isfinite(dqkv).all())
    if one:
        assert bool(torch.isnan(delta).all())
    else:
        want = (d_o.float() * o.float()).reshape(b, s, a, dh).sum(-1).transpose(1, 2)
        assert float((delta - want).abs().max()) < 1e-4 * math.sqrt(dh)
