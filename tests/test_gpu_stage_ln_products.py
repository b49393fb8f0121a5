"""fp32 stages whose LayerNorms go out with the product that reads their result: rows of one, two and up to four chunks of 16 per wave
(and some waves without one), token counts that fill no tile, one token, an FFN narrower than the rows (its LayerNorms have launches of
their own), both sides of the line on tiles x row length, recomputation (the copy of the input is the only one kept); the sums
of the small gradients in the launch of the weight gradients (up to four layers) and in one of their own (more)."""
import numpy as np
import pytest

from paper_2006_09503_amd import synth

from gpu_util import rel, run_stage_gpu, run_stage_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads,ffn,seq,micro,layers,recompute",
                         [(16, 1, 64, 1, 1, 1, 0), (64, 2, 256, 33, 1, 2, 0), (80, 2, 72, 17, 2, 3, 0), (128, 4, 512, 64, 2, 2, 1),
                          (144, 3, 576, 31, 1, 2, 0), (256, 4, 256, 50, 1, 2, 1), (272, 17, 1088, 15, 1, 2, 0), (512, 8, 520, 16, 1, 2, 0),
                          (528, 11, 528, 16, 1, 2, 0), (128, 2, 512, 260, 3, 2, 0), (128, 2, 512, 264, 4, 1, 0), (72, 1, 288, 20, 2, 2, 0), (48, 2, 96, 10, 1, 4, 0), (48, 2, 96, 10, 1, 5, 0)])
def test_layernorms_in_the_products_launch(hidden, heads, ffn, seq, micro, layers, recompute):
    cfg = synth.StageConfig(layers, hidden, heads, ffn, seq, micro, 2, 2, synth.MASK_PADDING if micro % 2 else synth.MASK_CAUSAL, synth.PREC_FP32,
                            recompute=recompute, min_len=1)
    gen = synth.StageInputs(cfg, 11)
    w0 = gen.weights()
    # gains and shifts that are no ones and zeros, and rows with a mean far from zero: the order of the operations shows
    for layer in synth.param_slices(cfg):
        for name in ("ln1_g", "ln1_b", "ln2_g", "ln2_b"):
            off, (n,) = layer[name]
            w0[off:off + n] += np.linspace(-0.5, 0.5, n, dtype=np.float32)
    mbs = [(x + 3.0, dy, lens) for x, dy, lens in gen.microbatches(2)]
    gpu = run_stage_gpu(cfg, w0, mbs, 2, two_streams=True)
    want = run_stage_oracle(cfg, w0, mbs)
    for k in want.Y:
        assert rel(gpu["Y"][k], want.Y[k]) < 5e-6 and rel(gpu["dX"][k], want.dX[k]) < 5e-6
    G = gpu["snaps"][0]["G"]
    for slices in synth.param_slices(cfg):
        for name, (off, shape) in slices.items():
            n = int(np.prod(shape))
            g, w = G[off:off + n], want.G[0][off:off + n]
            # (the key part of the QKV bias has a gradient of zero but for rounding: relative to the whole)
            assert np.abs(g - w).max() < 2e-5 * np.abs(w).max(), name


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("hidden,heads,seq,pos", [(16, 1, 20, 19), (128, 4, 20, 3), (272, 17, 20, 19), (512, 8, 33, 32)])
def test_infinities_and_nans_stay_with_their_tokens(hidden, heads, seq, pos, bad):
    """One token of the second of two sequences holds infinities or NaNs, in its input or in its output gradient: rows of the first sequence in
    the same tiles, and later or earlier tokens that a causal mask keeps apart, come out as without it.  (seq 20: the first 16 rows end
    inside the first sequence; pos = seq - 1: the row that the rows past the matrix are copies of.)"""
    cfg = synth.StageConfig(2, hidden, heads, 2 * hidden, seq, 2, 1, 1, synth.MASK_CAUSAL, synth.PREC_FP32)
    gen = synth.StageInputs(cfg, 7)
    w0 = gen.weights()
    x, dy, lens = gen.microbatches(1)[0]
    run = lambda x, dy: run_stage_gpu(cfg, w0, [(x, dy, lens)], 1, snapshot=False)
    clean = run(x, dy)
    px, pdy = x.copy(), dy.copy()
    px[1, pos] = bad
    pdy[1, pos] = bad
    got = run(px, dy)
    y, dx = got["Y"][1], got["dX"][1]
    assert np.array_equal(y[0], clean["Y"][1][0]) and np.array_equal(dx[0], clean["dX"][1][0])
    if pos > 0:
        assert rel(y[1, :pos], clean["Y"][1][1, :pos]) < 2e-6
    assert np.isnan(y[1, pos]).all()
    got = run(x, pdy)
    y, dx = got["Y"][1], got["dX"][1]
    assert np.array_equal(y, clean["Y"][1]) and np.array_equal(dx[0], clean["dX"][1][0])
    if pos + 1 < seq:
        assert rel(dx[1, pos + 1:], clean["dX"][1][1, pos + 1:]) < 2e-6
    assert np.isnan(dx[1, pos]).all()
