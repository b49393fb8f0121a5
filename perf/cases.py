"""Workloads whose speed is followed over time: the calls a user of this library makes, over the sizes, data types and
options that are used in earnest.  A case is a dict of plain values; `prepare` makes what a program has in hand before
the call, `run` is one pass through the public entry points (the C ABI as binding.py exposes it) and returns the
outputs, `work` the bytes and operations the pass cannot do without, `exact` the same outputs in 64 bits.

Kinds of cases:
  stage      whole 2BW training steps of one pipeline stage: three batches of m microbatches in 1F1B order, an update
             after each, as a pipeline worker drives the stage.  Outputs: every y and dx; the third batch runs on the
             weights the first batch's gradients made, so the coalesced gradients and the update show in them.  Stages
             small enough to be read back in passing return their weights and moments too.
  mlp        one block's feed-forward part: FC1 + GELU, FC2 + residual, then both data gradients, the FC1 bias gradient
             and both weight gradients, added to the coalesced accumulators.
  linear     one projection: forward with bias, data gradient, weight gradient added to the accumulator, bias gradient.
  attention  masked softmax attention of one microbatch, forward and backward, with the QKV bias gradient.
  norm       LayerNorm forward and backward with residual gradient, parameter gradients and column sums.
  update     the optimizer step on the coalesced gradient, with the bf16 copy of the new weights where bf16 trains.
"""
import math

import numpy as np
import torch

from paper_2006_09503_amd import binding as B
from paper_2006_09503_amd import synth

F32, BF16 = 0, 1
FUSED_DBIAS_HEADS = (32, 64, 80, 128)   # bf16 head sizes whose attention backward also returns the QKV bias gradient


def listed():
    return [
        # the parity configuration: tiny fp32 stage, everything is launch latency
        dict(name="stage_tiny_fp32", kind="stage", dtype=F32, layers=2, h=128, heads=4, f=512, s=64, b=2, m=4, inflight=2,
             mask=0, recompute=0),
        # a layer of the BERT-Large-shaped stage: 8 padded sequences of 512, bf16, two streams
        dict(name="stage_bert_bf16", kind="stage", dtype=BF16, layers=1, h=1024, heads=16, f=4096, s=512, b=8, m=4, inflight=4,
             mask=2, recompute=0),
        # feed-forward part of the h = 2560 GPT shape, 4 x 1024 tokens
        dict(name="mlp_gpt2560", kind="mlp", t=4096, h=2560, f=10240),
        # feed-forward part of the largest shape: one sequence of 2048 tokens, h = 8192
        dict(name="mlp_8192", kind="mlp", t=2048, h=8192, f=32768),
        # the QKV projection of one short sequence: few tokens against a full weight matrix
        dict(name="linear_short", kind="linear", dtype=BF16, t=128, n_in=1024, n_out=3072),
        # the QKV projection of 16 heads of 96 on 3 sequences of 1000 tokens: no size is a multiple of a tile
        dict(name="linear_ragged", kind="linear", dtype=BF16, t=3000, n_in=1536, n_out=4608),
        # attention of the BERT-Large-shaped stage, key padding
        dict(name="attn_bert", kind="attention", dtype=BF16, b=8, s=512, heads=16, dh=64, mask=2),
        # attention of the largest shape, causal
        dict(name="attn_8192", kind="attention", dtype=BF16, b=1, s=2048, heads=64, dh=128, mask=1),
        # 16 heads of 96, sequences of 1000 tokens, causal
        dict(name="attn_heads96", kind="attention", dtype=BF16, b=3, s=1000, heads=16, dh=96, mask=1),
        # fp32 attention, as the fp32 mode of a stage runs it
        dict(name="attn_fp32", kind="attention", dtype=F32, b=2, s=512, heads=8, dh=64, mask=1),
        # LayerNorm of the h = 2560 GPT shape
        dict(name="norm_2560", kind="norm", dtype=BF16, rows=4096, h=2560),
        # Adam on the parameters of the 6-layer BERT-Large-shaped stage, master weights and bf16 copy
        dict(name="update_adam", kind="update", n=75577344, adam=True, lp=True),
    ]


def _log(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, round(v / step) * step)))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "mlp", "mlp", "attention", "attention", "attention", "attention",
                       "norm", "update", "stage"])
    if kind == "linear":
        return dict(kind=kind, dtype=rng.choice([BF16, BF16, BF16, F32]), t=_log(rng, 32, 4096, 1), n_in=_log(rng, 128, 4096, 8),
                    n_out=_log(rng, 128, 8192, 8))
    if kind == "mlp":
        h = _log(rng, 256, 4096, 8)
        return dict(kind=kind, t=_log(rng, 128, 4096, 1), h=h, f=4 * h)
    if kind == "attention":
        dtype = rng.choice([BF16, BF16, BF16, F32])
        dh = rng.choice([32, 40, 48, 64, 64, 72, 80, 96, 96, 112, 128, 128])
        s = _log(rng, 48, 2048 if dtype == BF16 else 768, 1)
        heads = rng.choice([4, 8, 12, 16])
        return dict(kind=kind, dtype=dtype, b=rng.randint(1, max(1, min(8, 4096 // s))), s=s, heads=heads, dh=dh, mask=rng.randint(0, 2))
    if kind == "norm":
        return dict(kind=kind, dtype=rng.choice([BF16, BF16, F32]), rows=_log(rng, 64, 8192, 1), h=_log(rng, 128, 8192, 8))
    if kind == "update":
        return dict(kind=kind, n=_log(rng, 100000, 75000000, 4), adam=rng.random() < 0.7, lp=rng.random() < 0.7)
    heads, dh = rng.choice([2, 4, 8]), rng.choice([32, 48, 64])
    h = heads * dh
    return dict(kind="stage", dtype=rng.choice([F32, BF16]), layers=rng.randint(1, 2), h=h, heads=heads, f=4 * h, s=_log(rng, 32, 256, 1),
                b=rng.randint(1, 4), m=4, inflight=rng.choice([1, 2, 4]), mask=rng.randint(0, 2), recompute=rng.randint(0, 1))


# ----------------------------------------------------------------------------- inputs

BATCHES = 3            # batches of one pass of a stage: the third runs on the version the first one's gradients made
LR = 1e-4
LN_EPS = 1e-5
ADAM = dict(lr=LR, beta1=0.9, beta2=0.999, eps=1e-8)
UPDATE_M, UPDATE_STEP = 8, 100
READ_BACK = 1 << 20    # parameters up to which a stage's weights are part of a pass's outputs


def _tdt(dtype):
    return torch.bfloat16 if dtype == BF16 else torch.float32


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 2654435761 % (1 << 62) + 7)


def _rnd(g, shape, dtype, scale=1.0, shift=0.0):
    return (torch.randn(shape, generator=g, device="cuda") * scale + shift).to(_tdt(dtype))


def _empty(shape, dtype):
    return torch.empty(shape, device="cuda", dtype=_tdt(dtype))


def _lens(g, b, s):
    """Key lengths: three quarters of the sequence or more, as padded batches have."""
    return torch.randint(max(1, 3 * s // 4), s + 1, (b,), generator=g, device="cuda", dtype=torch.int32)


def _stage_config(c):
    return synth.StageConfig(c["layers"], c["h"], c["heads"], c["f"], c["s"], c["b"], c["m"], c["inflight"], c["mask"],
                             synth.PREC_BF16 if c["dtype"] == BF16 else synth.PREC_FP32, recompute=c["recompute"], lr=LR, ln_eps=LN_EPS)


def _inputs(c, seed):
    """The seeded tensors of a case, shared by `prepare` and `exact`."""
    g, k, dt = _gen(seed), c["kind"], c.get("dtype", BF16)
    if k == "stage":
        cfg = _stage_config(c)
        w = torch.randn(synth.param_count(cfg), generator=g, device="cuda") * 0.02
        for layer in synth.param_slices(cfg):
            for name in ("ln1_g", "ln2_g"):
                off, (n,) = layer[name]
                w[off:off + n] += 1.0
        w = w.to(_tdt(dt)).float()
        shape = (c["b"], c["s"], c["h"])
        mbs = []
        for _ in range(BATCHES * c["m"]):
            x, dy = _rnd(g, shape, dt), _rnd(g, shape, dt, 1e-2)
            lens = _lens(g, c["b"], c["s"]) if c["mask"] == 2 else None
            if lens is not None:   # no gradient arrives at padded positions
                dy *= (torch.arange(c["s"], device="cuda")[None, :] < lens[:, None])[..., None]
            mbs.append((x, lens, dy))
        return dict(cfg=cfg, w=w, mbs=mbs)
    if k == "mlp":
        t, h, f = c["t"], c["h"], c["f"]
        return dict(x=_rnd(g, (t, h), dt), w1=_rnd(g, (h, f), dt, 0.02), b1=_rnd(g, (f,), dt, 0.02), w2=_rnd(g, (f, h), dt, 0.02),
                    b2=_rnd(g, (h,), dt, 0.02), res=_rnd(g, (t, h), dt), dy=_rnd(g, (t, h), dt, 1e-2),
                    g1=_rnd(g, (h, f), F32, 0.1), gb1=_rnd(g, (f,), F32, 0.1), g2=_rnd(g, (f, h), F32, 0.1))
    if k == "linear":
        t, n, m = c["t"], c["n_in"], c["n_out"]
        return dict(x=_rnd(g, (t, n), dt), w=_rnd(g, (n, m), dt, 0.02), bias=_rnd(g, (m,), dt, 0.02), dy=_rnd(g, (t, m), dt, 1e-2),
                    gw=_rnd(g, (n, m), F32, 0.1), gb=_rnd(g, (m,), F32, 0.1))
    if k == "attention":
        b, s, h = c["b"], c["s"], c["heads"] * c["dh"]
        lens = _lens(g, b, s) if c["mask"] == 2 else None
        return dict(qkv=_rnd(g, (b, s, 3 * h), dt), do=_rnd(g, (b, s, h), dt), lens=lens)
    if k == "norm":
        r, h = c["rows"], c["h"]
        return dict(x=_rnd(g, (r, h), dt), gain=_rnd(g, (h,), dt, 0.02, 1.0), shift=_rnd(g, (h,), dt, 0.02),
                    dy=_rnd(g, (r, h), dt, 1e-2), dres=_rnd(g, (r, h), dt, 1e-2))
    n = c["n"]
    return dict(w=_rnd(g, (n,), F32, 0.02), m=_rnd(g, (n,), F32, 1e-3), v=_rnd(g, (n,), F32, 1e-3).square_(), g=_rnd(g, (n,), F32, 1e-2))


def prepare(case, seed):
    c = dict(case)
    st = _inputs(c, seed)
    st["case"] = c
    k, dt, L = c["kind"], c.get("dtype", BF16), B.lib()
    if k == "stage":
        cfg = st["cfg"]
        stage = B.Stage(cfg, st.pop("w").cpu().numpy(), stream=torch.cuda.current_stream())
        if cfg.recommended_streams == 2:
            st["bstream"] = torch.cuda.Stream()
            stage.set_backward_stream(st["bstream"])
        shape = (c["b"], c["s"], c["h"])
        n = BATCHES * c["m"]
        st.update(stage=stage, next_mb=1, y=[_empty(shape, dt) for _ in range(n)], dx=[_empty(shape, dt) for _ in range(n)])
        torch.cuda.synchronize()
    elif k == "mlp":
        t, h, f = c["t"], c["h"], c["f"]
        st.update(u=_empty((t, f), dt), a=_empty((t, f), dt), y=_empty((t, h), dt), du=_empty((t, f), dt), dx=_empty((t, h), dt),
                  ws=_empty((L.k2bw_gemm_dgrad_gelu_bias_workspace(t, f),), F32))
    elif k == "linear":
        t, n, m = c["t"], c["n_in"], c["n_out"]
        st.update(y=_empty((t, m), dt), dx=_empty((t, n), dt), ws=_empty((L.k2bw_bias_grad_workspace(m),), F32))
    elif k == "attention":
        b, s, a, dh = c["b"], c["s"], c["heads"], c["dh"]
        h = a * dh
        fused = dt == BF16 and dh in FUSED_DBIAS_HEADS
        ws = L.k2bw_attention_bwd_workspace(b, s, a, dh) if fused else L.k2bw_bias_grad_workspace(3 * h)
        st.update(fused=fused, o=_empty((b, s, h), dt), lse=_empty((b, a, s), F32), delta=_empty((b, a, s), F32),
                  dqkv=_empty((b, s, 3 * h), dt), db=_empty((3 * h,), F32), ws=_empty((ws,), F32))
    elif k == "norm":
        r, h = c["rows"], c["h"]
        st.update(y=_empty((r, h), dt), mean=_empty((r,), F32), rstd=_empty((r,), F32), dx=_empty((r, h), dt),
                  dgs=_empty((2 * h,), F32), dxs=_empty((h,), F32), ws=_empty((L.k2bw_layernorm_bwd_workspace(h),), F32))
    else:
        st["lp"] = _empty((c["n"],), BF16) if c["lp"] else None
    return st


# ----------------------------------------------------------------------------- one pass

def _ok(rc):
    B.check(rc, "perf case")


def run(st):
    c, L = st["case"], B.lib()
    dt = c.get("dtype", BF16)
    s_ = torch.cuda.current_stream().cuda_stream
    p = lambda name: st[name].data_ptr()   # noqa: E731
    if c["kind"] == "stage":
        first, n, stage = st["next_mb"], BATCHES * c["m"], st["stage"]
        stage.run_1f1b(first, n, lambda k: st["mbs"][k - first], lambda k: (st["y"][k - first], st["dx"][k - first]), c["inflight"])
        st["next_mb"] = first + n
        if "bstream" in st:
            torch.cuda.current_stream().wait_stream(st["bstream"])
        out = [st["y"], st["dx"]]
        if stage.n_params <= READ_BACK:
            out += [stage.read_weights(B.WEIGHTS_MASTER), *stage.read_adam()]
        return out
    if c["kind"] == "mlp":
        t, h, f = c["t"], c["h"], c["f"]
        _ok(L.k2bw_gemm(dt, 0, 0, 1, t, f, h, p("x"), h, p("w1"), f, p("u"), f, p("b1"), None, p("a"), 0, s_))
        _ok(L.k2bw_gemm(dt, 0, 0, 0, t, h, f, p("a"), f, p("w2"), h, p("y"), h, p("b2"), p("res"), None, 0, s_))
        _ok(L.k2bw_gemm_dgrad_gelu_bias(t, f, h, p("dy"), h, p("w2"), h, p("du"), f, p("u"), p("gb1"), 1, p("ws"), s_))
        _ok(L.k2bw_gemm(dt, 0, 1, 0, t, h, f, p("du"), f, p("w1"), f, p("dx"), h, None, None, None, 0, s_))
        _ok(L.k2bw_gemm(dt, 1, 0, 3, f, h, t, p("a"), f, p("dy"), h, p("g2"), h, None, None, None, 1, s_))
        _ok(L.k2bw_gemm(dt, 1, 0, 3, h, f, t, p("x"), h, p("du"), f, p("g1"), f, None, None, None, 1, s_))
        return [st[k] for k in ("u", "a", "y", "du", "dx", "gb1", "g1", "g2")]
    if c["kind"] == "linear":
        t, n, m = c["t"], c["n_in"], c["n_out"]
        _ok(L.k2bw_gemm(dt, 0, 0, 0, t, m, n, p("x"), n, p("w"), m, p("y"), m, p("bias"), None, None, 0, s_))
        _ok(L.k2bw_gemm(dt, 0, 1, 0, t, n, m, p("dy"), m, p("w"), m, p("dx"), n, None, None, None, 0, s_))
        _ok(L.k2bw_gemm(dt, 1, 0, 3, n, m, t, p("x"), n, p("dy"), m, p("gw"), m, None, None, None, 1, s_))
        _ok(L.k2bw_bias_grad(dt, t, m, p("dy"), p("gb"), 1, p("ws"), s_))
        return [st[k] for k in ("y", "dx", "gw", "gb")]
    if c["kind"] == "attention":
        b, s, a, dh = c["b"], c["s"], c["heads"], c["dh"]
        lens = None if st["lens"] is None else p("lens")
        _ok(L.k2bw_attention_fwd(dt, b, s, a, dh, c["mask"], lens, p("qkv"), p("o"), p("lse"), s_))
        fused = st["fused"]
        _ok(L.k2bw_attention_bwd(dt, b, s, a, dh, c["mask"], lens, p("qkv"), p("o"), p("lse"), p("do"), p("dqkv"), p("delta"),
                                 p("db") if fused else None, 0, p("ws") if fused else None, s_))
        if not fused:
            _ok(L.k2bw_bias_grad(dt, b * s, 3 * a * dh, p("dqkv"), p("db"), 0, p("ws"), s_))
        return [st[k] for k in ("o", "lse", "dqkv", "db")]
    if c["kind"] == "norm":
        r, h = c["rows"], c["h"]
        _ok(L.k2bw_layernorm_fwd(dt, r, h, LN_EPS, p("x"), p("gain"), p("shift"), p("y"), p("mean"), p("rstd"), s_))
        _ok(L.k2bw_layernorm_bwd(dt, r, h, p("dy"), p("x"), p("mean"), p("rstd"), p("gain"), p("dres"), p("dx"), p("dgs"), p("dxs"), 0,
                                 p("ws"), s_))
        return [st[k] for k in ("y", "mean", "rstd", "dx", "dgs", "dxs")]
    lp = None if st["lp"] is None else p("lp")
    if c["adam"]:
        _ok(L.k2bw_adam(c["n"], p("w"), p("w"), lp, p("m"), p("v"), p("g"), ADAM["lr"], ADAM["beta1"], ADAM["beta2"], ADAM["eps"], UPDATE_M,
                        UPDATE_STEP, s_))
    else:
        _ok(L.k2bw_momentum(c["n"], p("w"), p("w"), lp, p("m"), p("g"), ADAM["lr"], ADAM["beta1"], UPDATE_M, s_))
    return [st[k] for k in (("w", "m", "v") if c["adam"] else ("w", "m"))] + ([] if lp is None else [st["lp"]])


# ----------------------------------------------------------------------------- what a pass needs

def _attention_work(b, s, a, dh, mask, e):
    """Forward and backward: 2 + 5 products of s x s x dh per head; a causal mask leaves half of them."""
    pairs = s * (s + 1) / 2 if mask == 1 else s * s * (0.875 if mask == 2 else 1.0)
    h = a * dh
    return (b * s * (3 + 1) * h * e + b * s * (3 + 1 + 1 + 3) * h * e, 14.0 * b * pairs * h)


def work(case):
    c, k = case, case["kind"]
    e = 2 if c.get("dtype", BF16) == BF16 else 4
    if k == "stage":
        n, t, h, f = BATCHES * c["m"], c["b"] * c["s"], c["h"], c["f"]
        mat = 4 * h * h + 2 * h * f
        p = c["layers"] * (mat + 9 * h + f)
        by, fl = _attention_work(c["b"], c["s"], c["heads"], h // c["heads"], c["mask"], e)
        flops = n * c["layers"] * (6.0 * t * mat + fl)
        # boundary tensors of every microbatch, weights once per pass and direction, the update once per batch
        return dict(bytes=n * (4.0 * t * h * e + 2 * p * e) + BATCHES * p * (30 if e == 2 else 28), flops=flops)
    if k == "mlp":
        t, h, f = c["t"], c["h"], c["f"]
        # every operand once per pass: x, res, dy, y, dx; u, a, du written (u, a, du are saved for or read by other steps)
        return dict(bytes=5.0 * t * h * 2 + 3.0 * t * f * 2 + 2.0 * h * f * 2 + 2.0 * h * f * 8, flops=12.0 * t * h * f)
    if k == "linear":
        t, n, m = c["t"], c["n_in"], c["n_out"]
        return dict(bytes=e * (2.0 * t * n + 2.0 * t * m + n * m) + 8.0 * n * m, flops=6.0 * t * n * m)
    if k == "attention":
        by, fl = _attention_work(c["b"], c["s"], c["heads"], c["dh"], c["mask"], e)
        return dict(bytes=float(by), flops=fl)
    if k == "norm":
        return dict(bytes=e * 6.0 * c["rows"] * c["h"], flops=20.0 * c["rows"] * c["h"])
    return dict(bytes=c["n"] * ((28.0 if c["adam"] else 20.0) + (2.0 if c["lp"] else 0.0)), flops=12.0 * c["n"])


def tolerance(case):
    if case["kind"] == "update":
        return {"rel": 5e-5, "max": 0.02}    # a weight that differs in its last bit may fall on the other side of a bf16 tie
    if case.get("dtype", BF16) == F32:
        # Adam divides by the root of a moment that starts at zero: gradients at the rounding level decide a step's sign
        return {"rel": 2e-5, "max": 0.1} if case["kind"] == "stage" else {"rel": 1e-5}
    return {"rel": 1e-2, "max": 0.5}


# ----------------------------------------------------------------------------- the same in 64 bits

def _gelu(u):
    return u * 0.5 * (1.0 + torch.erf(u / math.sqrt(2.0)))


def _visible(mask, s, lens, n):
    i = torch.arange(s, device="cuda")
    if mask == 1:
        return i[None, :] <= i[:, None]
    return (i < int(lens[n]))[None, :].expand(s, s) if mask == 2 else torch.ones(s, s, dtype=torch.bool, device="cuda")


def _attention64(qkv, heads, mask, lens):
    """(o, lse) of [b, s, 3h] in 64 bits."""
    b, s, h3 = qkv.shape
    h = h3 // 3
    out, lse = [], []
    for n in range(b):
        q, k, v = (qkv[n, :, i * h:(i + 1) * h].reshape(s, heads, h // heads).transpose(0, 1).contiguous() for i in range(3))
        sc = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(h // heads)
        sc = sc.masked_fill(~_visible(mask, s, lens, n), -math.inf)
        out.append(torch.bmm(torch.softmax(sc, -1), v).transpose(0, 1).reshape(s, h))
        lse.append(torch.logsumexp(sc, -1))
    return torch.stack(out), torch.stack(lse)


def _norm64(x, g, s):
    mu = x.mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(((x - mu) ** 2).mean(-1, keepdim=True) + LN_EPS) * g + s


def _stage64(c, i):
    """Replay of the delayed updates: microbatch k on version max((k-1)//m - 1, 0), Adam on the mean gradient."""
    cfg, m = i["cfg"], c["m"]
    slices = synth.param_slices(cfg)
    w = i["w"].double()
    versions, mom, var = [w], torch.zeros_like(w), torch.zeros_like(w)
    ys, dxs = [], []
    for t in range(BATCHES):
        read = versions[max(t - 1, 0)].clone().requires_grad_(True)
        grad = torch.zeros_like(w)
        for x, lens, dy in i["mbs"][t * m:(t + 1) * m]:
            x = x.double().requires_grad_(True)
            z = x
            for sl in slices:
                q = {k: read[o:o + math.prod(sh)].reshape(sh) for k, (o, sh) in sl.items()}
                o, _ = _attention64(_norm64(z, q["ln1_g"], q["ln1_b"]) @ q["wqkv"] + q["bqkv"], c["heads"], c["mask"], lens)
                z = z + o @ q["wo"] + q["bo"]
                z = z + _gelu(_norm64(z, q["ln2_g"], q["ln2_b"]) @ q["w1"] + q["b1"]) @ q["w2"] + q["b2"]
            gx, gw = torch.autograd.grad(z, (x, read), dy.double())
            ys.append(z.detach()), dxs.append(gx)
            grad += gw
        f = lambda v: float(np.float32(v))   # noqa: E731 (the library takes its hyper-parameters as 32-bit floats)
        grad /= m
        b1, b2 = f(cfg.beta1), f(cfg.beta2)
        mom, var = b1 * mom + (1 - b1) * grad, b2 * var + (1 - b2) * grad ** 2
        versions.append(versions[-1] - f(cfg.lr) * (mom / (1 - b1 ** (t + 1))) / (torch.sqrt(var / (1 - b2 ** (t + 1))) + f(cfg.adam_eps)))
    out = [ys, dxs]
    return out + [versions[-1], mom, var] if w.numel() <= READ_BACK else out


def exact(case, seed):
    c = dict(case)
    i, k = _inputs(c, seed), c["kind"]
    if k == "stage":
        return _stage64(c, i)
    d = {n: v.double() for n, v in i.items() if isinstance(v, torch.Tensor) and n != "lens"}
    if k == "mlp":
        u = d["x"] @ d["w1"] + d["b1"]
        a = _gelu(u)
        y = d["res"] + a @ d["w2"] + d["b2"]
        dg = 0.5 * (1.0 + torch.erf(u / math.sqrt(2.0))) + u * torch.exp(-0.5 * u * u) / math.sqrt(2.0 * math.pi)
        du = (d["dy"] @ d["w2"].t().contiguous()) * dg
        return [u, a, y, du, du @ d["w1"].t().contiguous(), d["gb1"] + du.sum(0), d["g1"] + d["x"].t().contiguous() @ du,
                d["g2"] + a.t().contiguous() @ d["dy"]]
    if k == "linear":
        return [d["x"] @ d["w"] + d["bias"], d["dy"] @ d["w"].t().contiguous(), d["gw"] + d["x"].t().contiguous() @ d["dy"],
                d["gb"] + d["dy"].sum(0)]
    if k == "attention":
        qkv = d["qkv"].requires_grad_(True)
        o, lse = _attention64(qkv, c["heads"], c["mask"], i["lens"])
        (g,) = torch.autograd.grad(o, qkv, d["do"])
        return [o.detach(), lse.detach(), g, g.sum((0, 1))]
    if k == "norm":
        x, mu = d["x"].requires_grad_(True), d["x"].mean(-1)
        gain, shift = d["gain"].requires_grad_(True), d["shift"].requires_grad_(True)
        y = _norm64(x, gain, shift)
        gx, gg, gs = torch.autograd.grad(y, (x, gain, shift), d["dy"])
        gx = gx + d["dres"]
        return [y.detach(), mu.detach(), 1.0 / torch.sqrt(d["x"].detach().var(-1, unbiased=False) + LN_EPS), gx, torch.cat([gg, gs]), gx.sum(0)]
    f = lambda v: float(np.float32(v))   # noqa: E731
    b1, b2, g = f(ADAM["beta1"]), f(ADAM["beta2"]), d["g"] / UPDATE_M
    m = b1 * d["m"] + (1 - b1) * g
    if not c["adam"]:
        w = d["w"] - f(ADAM["lr"]) * m
        return [w, m] + ([w] if c["lp"] else [])
    v = b2 * d["v"] + (1 - b2) * g * g
    w = d["w"] - f(ADAM["lr"]) * (m / (1 - b1 ** UPDATE_STEP)) / (torch.sqrt(v / (1 - b2 ** UPDATE_STEP)) + f(ADAM["eps"]))
    return [w, m, v] + ([w] if c["lp"] else [])
