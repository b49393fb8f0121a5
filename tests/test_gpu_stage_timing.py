"""The timing report of a stage whose LayerNorms and small sums run in the launches of the products, and of one where they have their own:
classes, launches, FLOPs and bytes of one forward and one backward pass, and names of product kernels that are kernels of the library."""
import re

import pytest
import torch

from paper_2006_09503_amd import binding as B
from paper_2006_09503_amd import synth

from gpu_util import to_dev
from test_kernel_resources import built_kernels

pytestmark = pytest.mark.gpu


def report(cfg):
    gen = synth.StageInputs(cfg, 3)
    st = B.Stage(cfg, gen.weights())
    x, dy, _ = gen.microbatches(1)[0]
    X, DY = to_dev(x, cfg.precision), to_dev(dy, cfg.precision)
    Y, DX = torch.empty_like(X), torch.empty_like(X)
    torch.cuda.synchronize()
    st.timing_enable(True, 256)
    st.forward(1, X, None, Y)
    st.backward(1, DY, DX)
    kernels, classes = st.timing_collect_kernels(), st.timing_collect()
    st.close()
    return kernels, classes


@pytest.mark.parametrize("hidden,heads,ffn,seq,layers,fused", [(128, 4, 512, 128, 2, True), (256, 4, 512, 40, 1, True), (512, 8, 1024, 16, 2, True),
                                                               (528, 11, 1056, 16, 2, False), (72, 1, 288, 40, 2, False)])
def test_report_of_fused_launches(hidden, heads, ffn, seq, layers, fused):
    cfg = synth.StageConfig(layers, hidden, heads, ffn, seq, 1, 4, 1, synth.MASK_NONE, synth.PREC_FP32)
    kernels, classes = report(cfg)
    T, h, f, n = seq, hidden, ffn, layers
    products = 2.0 * T * (4 * h * h + 2 * h * f) * n          # of a forward pass; twice that in a backward pass
    for cls in ("gemm_fwd", "gemm_dgrad", "gemm_wgrad"):
        assert classes[cls]["flops"] == products, cls
    assert (classes["gemm_fwd"]["launches"], classes["gemm_dgrad"]["launches"]) == (4 * n, 4 * n)
    # a LayerNorm reads T x h numbers and writes as many forward, reads three times and writes once as many backward; the first one and
    # the top one write a copy, too; mean and rstd
    ln_fwd = 4.0 * T * h * (2 * 2 * n + 1) + 8.0 * T * 2 * n
    ln_bwd = 4.0 * T * h * (4 * 2 * n + 1) + 8.0 * T * 2 * n
    last = 4.0 * T * h * 4 + 8.0 * T                          # LN1 of the bottom layer has no product behind it
    got = {k: (classes[k]["launches"], classes[k]["bytes"]) for k in ("ln_fwd", "ln_bwd")}
    if fused:
        assert got == {"ln_fwd": (0, 0.0), "ln_bwd": (1, last)}
        assert classes["gemm_fwd"]["bytes"] == ln_fwd and classes["gemm_dgrad"]["bytes"] == ln_bwd - last
        assert classes["bias_grad"]["launches"] == 0 and classes["gemm_wgrad"]["launches"] == 1
        assert classes["gemm_wgrad"]["bytes"] >= 4.0 * T * (3 * h + f) * n     # dQKV and du are summed row by row
    else:
        assert got == {"ln_fwd": (2 * n, ln_fwd), "ln_bwd": (2 * n, ln_bwd)}
        assert classes["gemm_fwd"]["bytes"] == classes["gemm_dgrad"]["bytes"] == 0
    built = {re.search(r"gemm_\w+<[^>]*>|gemm_\w+", name).group(0) for name, _ in built_kernels(r"gemm_")}
    named = {k for k in kernels if k.startswith("gemm_")}
    assert named and named <= built, named - built
    # the instances of a fused stage are told apart: forward, with GELU, backward, and (where a layer has one below) with GELU'
    ln = [k for k in named if k.startswith("gemm_f32_ln_kernel")]
    assert len(ln) == (3 + (n > 1) if fused else 0), ln


@pytest.mark.parametrize("hidden,heads,tokens", [(128, 4, (64, 256, 1024, 2048, 4096)), (256, 4, (64, 512, 1024, 2048)), (72, 1, (64, 128, 512)),
                                                 (512, 8, (64, 256, 384, 1024))])
def test_second_gradient_buffer_only_where_a_launch_needs_it(hidden, heads, tokens):
    """Between two numbers of tokens the device bytes of a stage grow by as much per token, but for the buffer that the output projection's
    data gradient has for itself where it runs in LayerNorm's launch: that one appears and goes with the launch."""
    had, rest = [], []
    for T in tokens:
        cfg = synth.StageConfig(1, hidden, heads, 2 * hidden, T, 1, 1, 1, synth.MASK_NONE, synth.PREC_FP32)
        st = B.Stage(cfg, synth.StageInputs(cfg, 3).weights())
        dy = torch.zeros((1, T, hidden), device="cuda")
        y, dx = torch.empty_like(dy), torch.empty_like(dy)
        torch.cuda.synchronize()
        st.timing_enable(True, 64)
        st.forward(1, dy, None, y)
        st.backward(1, dy, dx)
        had.append(any(re.match(r"gemm_f32_ln_kernel<true, \d, true, 0>", k) for k in st.timing_collect_kernels()))
        rest.append(st.query(B.Q_BYTES_ALLOCATED) - (T * hidden * 4 if had[-1] else 0))
        st.close()
    per_token = [(rest[i + 1] - rest[i]) / (tokens[i + 1] - tokens[i]) for i in range(len(tokens) - 1)]
    assert len(set(per_token)) == 1, (had, per_token)
    assert had[0] == (hidden % 16 == 0) and not had[-1], had
