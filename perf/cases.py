"""The work whose speed counts: what a program that verifies drafts with this library has it do.

A program that serves a model quantises its weights once (`quantize`), then repeats verification steps over
M = 1 .. 32 candidate positions: either the whole weight stream as one launch (`step`), or decoder blocks out of
single calls (`block`; `layer` is the seven plain linears of one, `attention` its attention alone), and at the end the
vocabulary projection with the acceptance decision (`head`, greedy or at a temperature).  Shapes are those of the
repository's own configurations (Qwen3-8B and Qwen3-32B layer dimensions, vocabulary 151936, 8 positions = 7 drafts
and one bonus token) or generic ones.  Weights are fp32 ~ N(0, 0.02^2) (unit gain where linears feed linears),
activations bf16 ~ N(0, 1) with a few outlier channels; all inputs follow from the seed.

Each case is a dict of plain values; `prepare` makes its device buffers, `run` is one pass through
`paper_2603_01399_amd.binding`, `exact` the same in 64 bits with plain torch.
"""
import math

import torch

from paper_2603_01399_amd import binding as qb

EPS = 1e-6
THETA = 1.0e6
LAYER_8B = {"hidden": 4096, "q": 4096, "kv": 1024, "inter": 12288}
LAYER_32B = {"hidden": 5120, "q": 8192, "kv": 1024, "inter": 25600}
VOCAB = 151936


def listed():
    return [
        # the smallest call in use: one 1024 x 1024 linear, where launch and latency are everything
        {"name": "linear_1024_m8", "kind": "linear", "weights": "int8", "m": 8, "k": 1024, "n": 1024},
        # the seven linears of a decoder layer, int8 weights, a draft of 15 tokens
        {"name": "layer_8b_int8_m16", "kind": "layer", "weights": "int8", "m": 16, **LAYER_8B},
        # the same with int8 activations (smoothing vectors given), the default draft of 7 tokens
        {"name": "layer_8b_w8a8_m8", "kind": "layer", "weights": "w8a8", "m": 8, **LAYER_8B},
        # the same with 4-bit group-wise weights
        {"name": "layer_8b_int4_m8", "kind": "layer", "weights": "int4", "m": 8, **LAYER_8B},
        # the same with full-precision weights, a short odd draft: the verifier before quantisation
        {"name": "layer_8b_bf16_m5", "kind": "layer", "weights": "bf16", "m": 5, **LAYER_8B},
        # the widest draft on the largest layer shapes
        {"name": "layer_32b_int8_m32", "kind": "layer", "weights": "int8", "m": 32, **LAYER_32B},
        # a complete decoder block: norms, attention over 4096 cached positions, SwiGLU, residuals
        {"name": "block_8b_m8_ctx4096", "kind": "block", "m": 8, "ctx": 4096, **LAYER_8B},
        # attention alone over a long context of ragged length, ragged draft
        {"name": "attention_m5_ctx30011", "kind": "attention", "m": 5, "ctx": 30011, "heads": 32, "kv_heads": 8},
        # vocabulary projection and greedy acceptance
        {"name": "head_8b_greedy_m8", "kind": "head", "weights": "int8", "m": 8, "k": 4096, "v": VOCAB, "t": 0.0},
        # vocabulary projection and acceptance at a temperature
        {"name": "head_8b_sample_m8", "kind": "head", "weights": "int8", "m": 8, "k": 4096, "v": VOCAB, "t": 0.8},
        # the whole weight stream of a verification step as one launch: 36 layers and the vocabulary
        {"name": "step_8b_m8", "kind": "step", "weights": "int8", "m": 8, "layers": 36, "v": VOCAB, **LAYER_8B},
        # preparing one weight matrix when a model is loaded
        {"name": "quantize_int8_12288x4096", "kind": "quantize", "weights": "int8", "source": "f32", "n": 12288, "k": 4096},
    ]


def _log_int(rng, lo, hi, step=1):
    """A multiple of `step` in lo .. hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi // step * step, max(-(-lo // step) * step, int(round(v / step)) * step))


def _draw_layer(rng):
    hidden = _log_int(rng, 1024, 5120, 128)
    kv = 128 * rng.choice([2, 4, 8])
    return {"hidden": hidden, "q": kv * rng.choice([2, 4, 8]), "kv": kv,
            "inter": min(25600, _log_int(rng, 2 * hidden, 5 * hidden, 128))}


def draw(rng):
    kind = rng.choice(["linear", "linear", "layer", "layer", "block", "attention", "head", "step", "quantize"])
    weights = rng.choice(["int8", "int8", "w8a8", "int4", "bf16"])
    m = _log_int(rng, 1, 32)
    if kind == "linear":
        return {"kind": kind, "weights": weights, "m": m, "k": _log_int(rng, 128, 16384, 128 if weights == "int4" else 64),
                "n": _log_int(rng, 128, 16384, 16)}
    if kind == "layer":
        return {"kind": kind, "weights": weights, "m": m, **_draw_layer(rng)}
    if kind == "block":
        return {"kind": kind, "m": m, "ctx": _log_int(rng, 64, 16384), **_draw_layer(rng)}
    if kind == "attention":
        kv = rng.choice([2, 4, 8])
        return {"kind": kind, "m": m, "ctx": _log_int(rng, 64, 65536), "heads": kv * rng.choice([1, 2, 4, 8]), "kv_heads": kv}
    if kind == "head":
        t = rng.choice([0.0, 0.0, 0.6, 1.0])
        return {"kind": kind, "weights": "int8" if t else weights, "m": max(2, m), "k": _log_int(rng, 1024, 5120, 128),
                "v": _log_int(rng, 32000, VOCAB, 16), "t": t}
    if kind == "step":
        return {"kind": kind, "weights": rng.choice(["int8", "int8", "w8a8", "bf16"]), "m": max(2, min(16, m)),
                "layers": _log_int(rng, 2, 9), "v": _log_int(rng, 32000, VOCAB, 16), **_draw_layer(rng)}
    return {"kind": "quantize", "weights": rng.choice(["int8", "int8", "w8a8", "int4", "bf16"]),
            "source": rng.choice(["f32", "bf16"]), "n": _log_int(rng, 1024, 25600, 16), "k": _log_int(rng, 1024, 8192, 128)}


# ---------------------------------------------------------------------------------------------------- inputs

class _Inputs:
    """Draws a case's inputs on the GPU in a fixed order; prepare() and exact() see the same values."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed))

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32)

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.gen, device="cuda", dtype=torch.float32)

    def activations(self, m, k):
        x = self.normal(m, k)
        x[:, 17::331] *= 8.0
        return x.to(torch.bfloat16)

    def weight(self, n, k, std=0.02):
        return self.normal(n, k).mul_(std)

    def gamma(self, k):
        return (1.0 + 0.2 * self.normal(k)).to(torch.bfloat16)

    def smooth(self, k):
        return torch.exp2(self.uniform(k) * 2.0 - 1.0)

    def choice(self, n, count):
        return torch.randperm(n, generator=self.gen, device="cuda")[:count]


def _layer_linears(c):
    """(name of the input, K, N) of the seven linears: q, k, v, o, gate, up, down."""
    h, q, kv, i = c["hidden"], c["q"], c["kv"], c["inter"]
    return [("x", h, q), ("x", h, kv), ("x", h, kv), ("attn", q, h), ("x2", h, i), ("x2", h, i), ("act", i, h)]


def _pack(fmt, w, smooth=None):
    """What a program keeps of a weight matrix."""
    if fmt == "int8":
        return qb.quantize_weights(w)
    if fmt == "w8a8":
        return qb.quantize_weights_smoothed(w, smooth)
    if fmt == "int4":
        return (qb.quantize_weights_w4(w),)
    return (qb.pack_bf16_weights(w),)


def _bf16_empty(*shape):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda")


def _linear_state(fmt, x, w, smooth):
    m, k = x.shape
    n = w.shape[0]
    return {"fmt": fmt, "x": x, "n": n, "w": _pack(fmt, w, smooth), "smooth": smooth, "y": _bf16_empty(m, n),
            "ws": qb.make_workspace(m, n, k) if fmt in ("int8", "bf16") else None}


def _run_linear(s):
    fmt, x, n, y = s["fmt"], s["x"], s["n"], s["y"]
    if fmt == "int8":
        return qb.w8_linear(x, s["w"][0], s["w"][1], n, y=y, workspace=s["ws"])
    if fmt == "w8a8":
        return qb.w8a8_linear(x, s["w"][0], s["w"][1], n, smooth=s["smooth"], y=y)
    if fmt == "int4":
        return qb.w4_linear(x, s["w"][0], n, y=y)
    return qb.bf16_linear(x, s["w"][0], n, y=y, workspace=s["ws"])


def _linear_inputs(c, inp):
    """(fmt, x, w, smooth) of each linear of a `linear` or `layer` case, made one after the other."""
    fmt = c["weights"]
    if c["kind"] == "linear":
        shapes, widths = [("x", c["k"], c["n"])], {"x": c["k"]}
    else:
        shapes = _layer_linears(c)
        widths = {"x": c["hidden"], "attn": c["q"], "x2": c["hidden"], "act": c["inter"]}
    xs = {name: inp.activations(c["m"], k) for name, k in widths.items()}
    smooths = {name: inp.smooth(k) if fmt == "w8a8" else None for name, k in widths.items()}
    for name, k, n in shapes:
        yield fmt, xs[name], inp.weight(n, k), smooths[name]


def _plant(inp, w, h):
    """A clear winner per position, as a trained model has: raises one row's logit by 16.  Returns the rows."""
    t = inp.choice(w.shape[0], h.shape[0])
    h = h.float()
    w[t] += 16.0 * h / (h * h).sum(1, keepdim=True)
    return t


def _draft(inp, t, v):
    """Draft of len(t) - 1 tokens of which the first half agrees with the winners."""
    d = t[:-1].to(torch.int32)
    j = (d.numel() + 1) // 2
    d[j:] = (d[j:] + 1) % v
    return d.contiguous()


def _head_inputs(c, inp):
    h = inp.activations(c["m"], c["k"])
    smooth = inp.smooth(c["k"]) if c["weights"] == "w8a8" else None
    w = inp.weight(c["v"], c["k"])
    draft = _draft(inp, _plant(inp, w, h), c["v"])
    return h, smooth, w, draft, inp.uniform(c["m"]), inp.uniform(c["m"])


def _block_inputs(c, inp):
    m, h, q, kv, i, ctx = c["m"], c["hidden"], c["q"], c["kv"], c["inter"], c["ctx"]
    s = {"x": inp.activations(m, h), "g1": inp.gamma(h), "g2": inp.gamma(h), "qg": inp.gamma(128), "kg": inp.gamma(128)}
    s["k"] = inp.normal(ctx, kv // 128, 128).to(torch.bfloat16)
    s["v"] = inp.normal(ctx, kv // 128, 128).to(torch.bfloat16)
    s["wqkv"] = inp.weight(q + 2 * kv, h)
    s["wo"] = inp.weight(h, q)
    s["wgu"] = inp.weight(2 * i, h)          # rows in alternating blocks of 16: gate, up
    s["wdown"] = inp.weight(h, i)
    return s


def _attention_inputs(c, inp):
    m, hq, hk, ctx = c["m"], c["heads"], c["kv_heads"], c["ctx"]
    return {"qkv": inp.normal(m, (hq + 2 * hk) * 128).to(torch.bfloat16), "qg": inp.gamma(128), "kg": inp.gamma(128),
            "k": inp.normal(ctx, hk, 128).to(torch.bfloat16), "v": inp.normal(ctx, hk, 128).to(torch.bfloat16)}


def _cache(kv_heads, positions, k, v):
    cache = qb.KvCache(kv_heads, positions)
    cache.buf.zero_()
    cache.fill(k, v)
    return cache


def _step_inputs(c, inp):
    """Yields x0, then (w, smooth) of each linear in order, then the vocabulary's (w, smooth, draft).

    The linears feed each other (o reads q's output, gate and up read o's, down reads gate's, the next layer reads
    down's), so the winners of the vocabulary are planted at the hidden states that the unquantised chain ends in."""
    x = inp.activations(c["m"], c["hidden"])
    yield x
    a8 = c["weights"] == "w8a8"
    cur = x.float()
    for _ in range(c["layers"]):
        sm = {name: inp.smooth(k) if a8 else None
              for name, k in (("x", c["hidden"]), ("attn", c["q"]), ("x2", c["hidden"]), ("act", c["inter"]))}
        for i, (name, k, n) in enumerate(_layer_linears(c)):
            w = inp.weight(n, k, k ** -0.5)
            if i in (0, 3, 4, 6):
                cur = cur @ w.t()
            yield w, sm[name]
            del w
    smooth = inp.smooth(c["hidden"]) if a8 else None
    w = inp.weight(c["v"], c["hidden"])
    draft = _draft(inp, _plant(inp, w, cur), c["v"])
    yield w, smooth, draft


# ---------------------------------------------------------------------------------------------------- prepare and run

def prepare(case, seed):
    c, inp = case, _Inputs(seed)
    kind, fmt = c["kind"], c.get("weights")
    if kind in ("linear", "layer"):
        return {"kind": kind, "linears": [_linear_state(*a) for a in _linear_inputs(c, inp)]}
    if kind == "quantize":
        w = inp.weight(c["n"], c["k"])
        w = w.to(torch.bfloat16) if c["source"] == "bf16" else w
        smooth = inp.smooth(c["k"]) if fmt == "w8a8" else None
        return {"kind": kind, "fmt": fmt, "source": w, "smooth": smooth}
    if kind == "head":
        h, smooth, w, draft, ua, us = _head_inputs(c, inp)
        s = {"kind": kind, "fmt": fmt, "t": c["t"], "v": c["v"], "h": h, "smooth": smooth, "draft": draft, "ua": ua, "us": us}
        s["w"] = _pack(fmt, w, smooth)
        if c["t"]:
            s["ws"] = torch.empty(max(qb.lib().quasar_sample_workspace_bytes(c["m"], c["v"]), 16), dtype=torch.uint8, device="cuda")
        else:
            s["ws"] = qb.make_workspace(c["m"], c["v"], c["k"])
        return s
    if kind == "attention":
        a = _attention_inputs(c, inp)
        total = c["ctx"] + c["m"]
        return {"kind": kind, "heads": c["heads"], "ctx": c["ctx"], "total": total, "qkv": a["qkv"], "qg": a["qg"], "kg": a["kg"],
                "cache": _cache(c["kv_heads"], total, a["k"], a["v"]), "q": _bf16_empty(c["m"], c["heads"] * 128),
                "out": _bf16_empty(c["m"], c["heads"] * 128),
                "ws": qb.attention_workspace(c["m"], c["heads"], c["kv_heads"], total)}
    if kind == "block":
        a = _block_inputs(c, inp)
        m, heads, kv_heads, total = c["m"], c["q"] // 128, c["kv"] // 128, c["ctx"] + c["m"]
        s = {"kind": kind, "c": dict(c), "heads": heads, "total": total}
        s.update({n: a[n] for n in ("x", "g1", "g2", "qg", "kg")})
        s.update({n: _pack("int8", a[n]) for n in ("wqkv", "wo", "wgu", "wdown")})
        s["cache"] = _cache(kv_heads, total, a["k"], a["v"])
        s["ws"] = qb.attention_workspace(m, heads, kv_heads, total)
        for n, width in (("qkv", c["q"] + 2 * c["kv"]), ("q", c["q"]), ("attn", c["q"]), ("h1", c["hidden"]), ("act", c["inter"]),
                         ("h2", c["hidden"])):
            s[n + "_out"] = _bf16_empty(m, width)
        return s
    # step: the chain of linears and the vocabulary as one prepared launch
    m = c["m"]
    made = _step_inputs(c, inp)
    x = next(made)
    widths = [n for _, _, n in _layer_linears(c)]
    flat = _bf16_empty(c["layers"], m * sum(widths))          # every linear's output, [m, n] one after the other
    linears, smooths, cur = [], [], x
    for layer in range(c["layers"]):
        at, ys = 0, []
        for n in widths:
            ys.append(flat[layer, at:at + m * n].view(m, n))
            at += m * n
        xs = (cur, cur, cur, ys[0], ys[3], ys[3], ys[4])
        for i, n in enumerate(widths):
            w, smooth = next(made)
            packed = _pack(fmt, w, smooth)
            del w
            linears.append((xs[i], packed[0], packed[1] if len(packed) > 1 else None, n, ys[i]))
            smooths.append(smooth)
        cur = ys[6]
    w, smooth, draft = next(made)
    packed = _pack(fmt, w, smooth)
    del w
    argmax = torch.empty(m, dtype=torch.int32, device="cuda")
    accept = torch.empty(1, dtype=torch.int32, device="cuda")
    verify = (cur, packed[0], packed[1] if len(packed) > 1 else None, c["v"], draft, argmax, accept)
    seq = qb.Sequence(linears, verify, w8a8=True, smooth=smooths, verify_smooth=smooth) if fmt == "w8a8" else qb.Sequence(linears, verify)
    return {"kind": kind, "seq": seq, "y": flat, "argmax": argmax, "accept": accept}


def run(state):
    s = state
    kind = s["kind"]
    if kind in ("linear", "layer"):
        return [_run_linear(a) for a in s["linears"]]
    if kind == "quantize":
        return _pack(s["fmt"], s["source"], s["smooth"])
    if kind == "head":
        if s["t"]:
            return qb.lmhead_verify_sample(s["h"], *s["w"], s["v"], s["draft"], s["t"], s["ua"], s["us"], s["ws"])
        if s["fmt"] == "int8":
            return qb.lmhead_verify(s["h"], *s["w"], s["v"], s["draft"], s["ws"])
        if s["fmt"] == "w8a8":
            return qb.w8a8_lmhead_verify(s["h"], *s["w"], s["v"], s["draft"], s["ws"], smooth=s["smooth"])
        if s["fmt"] == "int4":
            return qb.w4_lmhead_verify(s["h"], *s["w"], s["v"], s["draft"], s["ws"])
        return qb.bf16_lmhead_verify(s["h"], *s["w"], s["v"], s["draft"], s["ws"])
    if kind == "attention":
        q = qb.attn_prepare(s["qkv"], s["heads"], s["cache"], s["ctx"], s["qg"], s["kg"], eps=EPS, rope_theta=THETA, q_out=s["q"])
        out = qb.verify_attention(q, s["heads"], s["cache"], s["total"], workspace=s["ws"], out=s["out"])
        return {"q": q, "out": out, "cache": s["cache"].buf}
    if kind == "block":
        c = s["c"]
        qkv = qb.w8_linear_fused(s["x"], *s["wqkv"], c["q"] + 2 * c["kv"], gamma=s["g1"], eps=EPS, y=s["qkv_out"])
        q = qb.attn_prepare(qkv, s["heads"], s["cache"], c["ctx"], s["qg"], s["kg"], eps=EPS, rope_theta=THETA, q_out=s["q_out"])
        attn = qb.verify_attention(q, s["heads"], s["cache"], s["total"], workspace=s["ws"], out=s["attn_out"])
        h1 = qb.w8_linear_fused(attn, *s["wo"], c["hidden"], residual=s["x"], y=s["h1_out"])
        act = qb.w8_gateup_swiglu(h1, *s["wgu"], c["inter"], gamma=s["g2"], eps=EPS, y=s["act_out"])
        h2 = qb.w8_linear_fused(act, *s["wdown"], c["hidden"], residual=h1, y=s["h2_out"])
        return {"qkv": qkv, "q": q, "attn": attn, "h1": h1, "act": act, "h2": h2, "cache": s["cache"].buf}
    s["seq"].run()
    return {"y": s["y"], "argmax": s["argmax"], "accept": s["accept"]}


# ---------------------------------------------------------------------------------------------------- bytes and tolerances

def _weight_bytes(fmt, n, k):
    """Codes and step sizes of one packed matrix."""
    if fmt == "int4":
        return n * k // 2 + 2 * n * (k // 128)
    return 2 * n * k if fmt == "bf16" else n * k + 2 * n


def work(case):
    c = case
    kind, m, fmt = c["kind"], c.get("m", 0), c.get("weights", "int8")

    def linears(shapes, inputs):
        b = sum(_weight_bytes(fmt, n, k) + 2 * m * n for k, n in shapes) + sum(2 * m * k for k in inputs)
        return b + (sum(4 * k for k in inputs) if fmt == "w8a8" else 0), sum(2 * m * n * k for k, n in shapes)

    def attention(heads, kv_heads, ctx):
        total = ctx + m
        b = 2 * total * kv_heads * 256 + 2 * m * heads * 256 + m * (heads + 2 * kv_heads) * 256
        return b, 4 * m * heads * 128 * total

    if kind == "linear":
        b, f = linears([(c["k"], c["n"])], [c["k"]])
    elif kind == "layer":
        b, f = linears([(k, n) for _, k, n in _layer_linears(c)], [c["hidden"], c["q"], c["hidden"], c["inter"]])
    elif kind == "quantize":
        b = c["n"] * c["k"] * (4 if c["source"] == "f32" else 2) + _weight_bytes(fmt, c["n"], c["k"])
        f = 0
    elif kind == "head":
        b, f = linears([(c["k"], c["v"])], [c["k"]])
        b -= 2 * m * c["v"]                                   # no logits leave the call
    elif kind == "attention":
        b, f = attention(c["heads"], c["kv_heads"], c["ctx"])
    elif kind == "block":
        h, q, kv, i = c["hidden"], c["q"], c["kv"], c["inter"]
        b, f = linears([(h, q + 2 * kv), (q, h), (h, 2 * i), (i, h)], [h, q, h, i])
        b2, f2 = attention(q // 128, kv // 128, c["ctx"])
        b, f = b + b2 - 2 * m * i, f + f2                     # gate and up leave as one product
    else:
        one = [(k, n) for _, k, n in _layer_linears(c)]
        b, f = linears(one * c["layers"] + [(c["hidden"], c["v"])], [c["hidden"], c["q"], c["hidden"], c["inter"]] * c["layers"] + [c["hidden"]])
        b -= 2 * m * c["v"]
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    c = case
    if c["kind"] == "quantize":
        return "exact"
    if c["kind"] == "head":
        # argmax and accepted length are whole values; probabilities are fp32 sums over the vocabulary
        return {"rel": 1e-5} if c["t"] else "exact"
    if c["kind"] == "step":
        return {"rel": 3e-2, "max": 0.5}    # bf16 roundings travel through the chain of linears: 1.4e-2 from exact()
    # bf16 outputs, distance from exact(): 5.5e-3 (block), 3.6e-3 (attention), 1.7e-3 (one linear); a new cache row may
    # differ in the last place
    if c["kind"] in ("block", "attention"):
        return {"rel": 2e-2 if c["kind"] == "block" else 1.2e-2, "max": 0.1, "differ": 2e-3}
    return {"rel": 6e-3, "max": 0.05}


# ---------------------------------------------------------------------------------------------------- the same in 64 bits

def _codes8(w, smooth=None):
    """fp32 or bf16 weights -> (integer codes as fp32, bf16 step sizes): one step size per row."""
    w = w.float()
    w = w / smooth if smooth is not None else w
    d = (w.abs().amax(1) / 127.0).to(torch.bfloat16)
    q = torch.clamp(torch.round(w / d.float()[:, None]), -127, 127)
    return torch.where(d.float()[:, None] > 0, q, torch.zeros_like(q)), d


def _codes4(w):
    """fp32 or bf16 weights -> (codes [n, k / 128, 128] as fp32, bf16 step sizes [n, k / 128])."""
    w = w.float().view(w.shape[0], -1, 128)
    d = (w.abs().amax(2) / 7.0).to(torch.bfloat16)
    q = torch.clamp(torch.round(w / d.float()[..., None]), -7, 7)
    return torch.where(d.float()[..., None] > 0, q, torch.zeros_like(q)), d


def _exact_linear(fmt, x, w, smooth, rows=16384):
    """x [m, k] in 64 bits times the quantised weights, [m, n] in 64 bits."""
    x = x.double()
    if fmt == "w8a8":
        xs = x.float() * smooth
        amax = xs.abs().amax(1, keepdim=True)
        codes = torch.clamp(torch.round(xs * (127.0 / amax)), -127, 127)
        x = codes.double() * (amax / 127.0).double()
    out = []
    for at in range(0, w.shape[0], rows):
        part = w[at:at + rows]
        if fmt in ("int8", "w8a8"):
            q, d = _codes8(part, smooth if fmt == "w8a8" else None)
            out.append((x @ q.double().t()) * d.double())
        elif fmt == "int4":
            q, d = _codes4(part)
            out.append(x @ (q.double() * d.double()[..., None]).reshape(part.shape[0], -1).t())
        else:
            out.append(x @ part.to(torch.bfloat16).double().t())
    return torch.cat(out, 1)


def _exact_norm(x, gamma):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + float(torch.tensor(EPS, dtype=torch.float32))) * gamma.double()


def _exact_rotary(x, pos):
    """x [m, heads, 128] at positions pos [m]."""
    i = torch.arange(64, device=x.device, dtype=torch.float64)
    angle = pos.double()[:, None] * THETA ** (-2.0 * i / 128.0)
    c, s = torch.cos(angle)[:, None], torch.sin(angle)[:, None]
    a, b = x[..., :64], x[..., 64:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _exact_attention(qkv, heads, kv_heads, ctx, qg, kg, k_cached, v_cached):
    """qkv [m, (heads + 2 kv_heads) 128] in 64 bits -> (queries, outputs), both [m, heads 128]."""
    m = qkv.shape[0]
    x = qkv.view(m, heads + 2 * kv_heads, 128)
    pos = torch.arange(ctx, ctx + m, device=qkv.device)
    q = _exact_rotary(_exact_norm(x[:, :heads], qg), pos)
    kn = _exact_rotary(_exact_norm(x[:, heads:heads + kv_heads], kg), pos)
    k = torch.cat([k_cached.double(), kn])
    v = torch.cat([v_cached.double(), x[:, heads + kv_heads:]])
    hidden_from = torch.arange(ctx + m, device=qkv.device)[None] > pos[:, None]
    out = torch.empty(m, heads, 128, dtype=torch.float64, device=qkv.device)
    group = heads // kv_heads
    for h in range(heads):
        s = q[:, h] @ k[:, h // group].t() / math.sqrt(128.0)
        out[:, h] = torch.softmax(s.masked_fill(hidden_from, -math.inf), -1) @ v[:, h // group]
    return q.reshape(m, -1), out.reshape(m, -1)


def _exact_pack8(q, d):
    n, k = q.shape
    tiles = q.to(torch.int8).view(n // 16, 16, k // 64, 4, 16)        # tile, row, step, group of 16 k, k
    return tiles.permute(0, 2, 3, 1, 4).contiguous().view(-1), d


def exact(case, seed):
    c, inp = case, _Inputs(seed)
    kind, fmt = c["kind"], c.get("weights")
    if kind in ("linear", "layer"):
        return [_exact_linear(f, x, w, smooth) for f, x, w, smooth in _linear_inputs(c, inp)]
    if kind == "quantize":
        w = inp.weight(c["n"], c["k"])
        w = w.to(torch.bfloat16) if c["source"] == "bf16" else w
        if fmt in ("int8", "w8a8"):
            return _exact_pack8(*_codes8(w, inp.smooth(c["k"]) if fmt == "w8a8" else None))
        return None
    if kind == "head":
        h, smooth, w, draft, ua, us = _head_inputs(c, inp)
        logits = _exact_linear(fmt, h, w, smooth)
        if not c["t"]:
            argmax = logits.argmax(1).int()
            hit = (argmax[:-1] == draft).int()
            return argmax, hit.cumprod(0).sum().int().view(1)
        p = torch.softmax(logits / c["t"], 1)
        return None, None, p.gather(1, torch.cat([draft, draft[-1:]]).long()[:, None])[:-1, 0]
    if kind == "attention":
        a = _attention_inputs(c, inp)
        q, out = _exact_attention(a["qkv"].double(), c["heads"], c["kv_heads"], c["ctx"], a["qg"], a["kg"], a["k"], a["v"])
        return {"q": q, "out": out, "cache": None}
    if kind == "block":
        a = _block_inputs(c, inp)
        x = a["x"].double()
        qkv = _exact_linear("int8", _exact_norm(x, a["g1"]), a["wqkv"], None)
        q, attn = _exact_attention(qkv, c["q"] // 128, c["kv"] // 128, c["ctx"], a["qg"], a["kg"], a["k"], a["v"])
        h1 = x + _exact_linear("int8", attn, a["wo"], None)
        gu = _exact_linear("int8", _exact_norm(h1, a["g2"]), a["wgu"], None).view(c["m"], c["inter"] // 16, 2, 16)
        act = (torch.nn.functional.silu(gu[:, :, 0]) * gu[:, :, 1]).reshape(c["m"], -1)
        h2 = h1 + _exact_linear("int8", act, a["wdown"], None)
        return {"qkv": qkv, "q": q, "attn": attn, "h1": h1, "act": act, "h2": h2, "cache": None}
    made = _step_inputs(c, inp)
    cur = next(made).double()
    ys = []
    for _ in range(c["layers"]):
        layer = []
        for i in range(7):
            x = cur if i < 3 else layer[{3: 0, 4: 3, 5: 3, 6: 4}[i]]
            layer.append(_exact_linear(fmt, x, *next(made)))
        cur = layer[6]
        ys.append(torch.cat([y.reshape(-1) for y in layer]))
    w, smooth, draft = next(made)
    argmax = _exact_linear(fmt, cur, w, smooth).argmax(1).int()
    return {"y": torch.stack(ys), "argmax": argmax, "accept": (argmax[:-1] == draft).int().cumprod(0).sum().int().view(1)}
