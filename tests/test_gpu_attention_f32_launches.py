"""fp32 attention, backward in one launch and in two: sizes on both sides of that rule, on one and on four waves per workgroup (all
four forms at heads above 64), head sizes of every row width in LDS; forward
with one workgroup per CU at a time; and what a position that nobody may see holds must not show in either form."""
import pytest
import torch

from test_gpu_attention_shapes import F32, TOL, inputs, reference, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [8, 24, 48, 64, 80, 104, 128])
@pytest.mark.parametrize("b,s,a,mask", [(1, 65, 2, 1), (2, 290, 8, 0), (2, 290, 8, 2), (2, 290, 8, 1), (2, 250, 9, 2), (9, 97, 30, 1), (40, 33, 13, 2),
                                        (3, 520, 24, 2), (4, 60, 72, 0), (13, 100, 12, 0), (19, 108, 16, 0), (2, 430, 10, 1), (1, 300, 32, 1)])
def test_backward_on_both_sides_of_the_launch_rule(dh, b, s, a, mask):
    h = a * dh
    qkv, d_o, lens = inputs(F32, b, s, a, dh, mask)
    o, lse, dqkv = run(F32, b, s, a, dh, mask, qkv, d_o, lens)
    o64, lse64, d64 = reference(qkv, d_o, a, mask, lens)
    tol = TOL[F32] * max(1.0, (s / 200) ** 0.5)   # (TOL is for sums of up to 200 rows)
    assert float((o.double() - o64).norm() / o64.norm()) < tol
    assert float((lse.double() - lse64).abs().max()) < 1e-5
    size = max(float(t.norm()) for t in d64.split(h, -1))
    for got, want in zip(dqkv.split(h, -1), d64.split(h, -1)):
        assert float((got.double() - want).norm()) < 2 * tol * size


@pytest.mark.parametrize("dh", [16, 40, 64, 96, 128])
@pytest.mark.parametrize("b,s,a,pos", [(1, 100, 2, 40), (2, 300, 8, 170), (36, 70, 16, 37)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_what_nobody_sees_does_not_show(dh, b, s, a, pos, bad):
    h = a * dh
    qkv, d_o, _ = inputs(F32, b, s, a, dh, 1)
    o0, lse0, d0 = run(F32, b, s, a, dh, 1, qkv, d_o, None)
    same = lambda x, y: bool(torch.isfinite(x).all()) and float((x - y).norm() / y.norm()) < 2e-6
    poisoned = qkv.clone()
    poisoned[:, pos, h:] = bad                       # K and V of one token
    o1, lse1, d1 = run(F32, b, s, a, dh, 1, poisoned, d_o, None)
    assert same(o1[:, :pos], o0[:, :pos]) and same(lse1[..., :pos], lse0[..., :pos]) and same(d1[:, :pos, :h], d0[:, :pos, :h])
    poisoned = d_o.clone()
    poisoned[:, pos] = bad                           # the gradient of one query
    _, _, d2 = run(F32, b, s, a, dh, 1, qkv, poisoned, None)
    assert same(d2[:, pos + 1:, h:], d0[:, pos + 1:, h:])
    lens = torch.full((b,), pos, device="cuda", dtype=torch.int32)
    o3, lse3, d3 = run(F32, b, s, a, dh, 2, qkv, d_o, lens)
    poisoned = qkv.clone()
    poisoned[:, pos:, h:] = bad                      # keys past the length
    o4, lse4, d4 = run(F32, b, s, a, dh, 2, poisoned, d_o, lens)
    assert torch.equal(o3, o4) and torch.equal(lse3, lse4) and torch.equal(d3, d4)
