"""The work that a user of this framework has it do, as cases to be timed and
compared: lone projections, stacks of projections (dependent decoder layers and
independent ones) and the loading of weights, each through the binding's public
calls (paper_2607_02501_amd.eb).

Sizes are those of the synthetic workloads in paper_2607_02501_amd/workloads.py
(a 7B-class decoder at one token, a flow-matching action expert at 50 rows, a
VLM prefill of 816 rows, a video backbone of 4096 rows), of the GPU tests'
ragged shapes, or generic ones between them.

A control tick (eb.multirate_tick) runs the stacks below one after another
and adds no device work of its own, so it is not a case of its own.

Every case is a dict with "kind":
  linear  one eb.qlinear_fused call (prologue, epilogue, path as given)
  chain   decoder layers, each QKV(norm(h)) -> O + h -> gated gate/up(norm(h))
          -> down + h, as one eb.qlinear_stack call over the fp32 stream h
  layers  independent projections as one eb.qlinear_stack call
  load    fp32 weights -> blocks, blocks -> canonical bytes -> blocks
"""
from __future__ import annotations

import torch

from paper_2607_02501_amd import eb

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
CODE_BITS = {"q8_0": 8.5, "q4_0": 4.5, "q6_s": 6.5625}
EPS = 1e-5


def listed():
    return [
        # one projection of a small policy head, one token: the smallest call there is
        dict(name="linear_1x2048_q8", kind="linear", qtype="q8_0", m=1, n=2048, k=2048, x="f16",
             y="f32", pro="", epi="", path="auto"),
        # a feed-forward projection for four robots (or four speculated tokens) at once
        dict(name="linear_4x11008_q4", kind="linear", qtype="q4_0", m=4, n=11008, k=4096, x="f16",
             y="f16", pro="", epi="", path="auto"),
        # a ragged projection: rows, columns and blocks that fill no tile of any kernel
        dict(name="linear_77x3001_q8", kind="linear", qtype="q8_0", m=77, n=3001, k=1504, x="bf16",
             y="bf16", pro="", epi="", path="auto"),
        # the gated feed-forward of the VLM prefill on the int8 path a caller may choose
        dict(name="linear_816x32768_q8_int8", kind="linear", qtype="q8_0", m=816, n=32768, k=2048,
             x="bf16", y="bf16", pro="", epi="glu", path="mfma_i8"),
        # one decoded token through the whole 7B-class backbone, 4-bit weights: a whole call
        dict(name="chain_decode_7b_q4", kind="chain", qtype="q4_0", m=1, d=4096, nqkv=12288,
             ff=11008, layers=32, x="f16"),
        # the same decoder in 6-bit weights, eight of its layers (more than the last-level cache)
        dict(name="chain_decode_7b_q6", kind="chain", qtype="q6_s", m=1, d=4096, nqkv=12288,
             ff=11008, layers=8, x="f16"),
        # one denoising step of the action expert, all 18 layers: a whole call
        dict(name="chain_expert_50_q8", kind="chain", qtype="q8_0", m=50, d=1024, nqkv=2048,
             ff=4096, layers=18, x="bf16"),
        # image and text tokens through four layers of the VLM backbone
        dict(name="chain_prefill_816_q8", kind="chain", qtype="q8_0", m=816, d=2048, nqkv=2560,
             ff=16384, layers=4, x="bf16"),
        # independent one-token projections (128 distinct matrices, as many small heads would have)
        dict(name="layers_128x2048_q8", kind="layers", qtype="q8_0", m=1, count=128,
             shapes="2048x2048", x="f16", y="f32"),
        # the action expert's projections of four layers, independent of each other
        dict(name="layers_expert_50_q8", kind="layers", qtype="q8_0", m=50, count=4,
             shapes="1024x2048,1024x1024,1024x8192,4096x1024", x="bf16", y="f32"),
        # one layer's projections of the video backbone: the most rows
        dict(name="layers_video_4096_q4", kind="layers", qtype="q4_0", m=4096, count=1,
             shapes="3072x9216,3072x3072,3072x12288,12288x3072", x="bf16", y="f32"),
        # loading a checkpoint matrix: quantize, export to block files' bytes, import again
        dict(name="load_11008x4096_q4", kind="load", qtype="q4_0", n=11008, k=4096),
    ]


# ---------------------------------------------------------------------------
# drawn cases
# ---------------------------------------------------------------------------

def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _mult(v, q):
    return max(q, (v + q // 2) // q * q)


def _one(rng, *choices):
    return choices[rng.randrange(len(choices))]


def draw(rng):
    kind = _one(rng, "linear", "linear", "linear", "chain", "chain", "layers", "layers", "load")
    qtype = _one(rng, "q8_0", "q4_0", "q6_s")
    kq = 256 if qtype == "q6_s" else 32
    x = _one(rng, "f16", "bf16")
    if kind == "linear":
        m, n, k = _log(rng, 1, 1024), _log(rng, 300, 16384), _mult(_log(rng, 256, 8192), kq)
        path, pro, epi = "auto", _one(rng, "", "", "rmsnorm"), _one(rng, "", "add", "glu")
        if qtype != "q6_s" and m >= 64 and rng.random() < 0.3:
            path, pro = "mfma_i8", ""
        while 2 * m * n * k > (40e9 if path == "mfma_i8" else 120e9):
            m = (m + 1) // 2
        if epi == "glu":
            n += n % 2
        return dict(kind=kind, qtype=qtype, m=m, n=n, k=k, x=x, y=_one(rng, "f32", "f16", "bf16"),
                    pro=pro, epi=epi, path=path)
    if kind == "chain":
        m, d = _one(rng, 1, _log(rng, 2, 128), _log(rng, 129, 1024)), _mult(_log(rng, 768, 4096), 256)
        ff = _mult(int(d * (2.5 + 2 * rng.random())), 256)
        nqkv, layers = d + 2 * _mult(d // _one(rng, 1, 4, 8), 64), 1 + rng.randrange(8)
        while layers > 1 and 2 * m * layers * (d * nqkv + d * d + 3 * d * ff) > 120e9:
            layers -= 1
        return dict(kind=kind, qtype=qtype, m=m, d=d, nqkv=nqkv, ff=ff, layers=layers, x=x)
    if kind == "layers":
        m, count = _one(rng, 1, _log(rng, 2, 128), _log(rng, 129, 2048)), 1 + rng.randrange(8)
        shapes = [(_mult(_log(rng, 512, 8192), kq), _log(rng, 512, 8192)) for _ in range(1 + rng.randrange(4))]
        while count > 1 and 2 * m * count * sum(a * b for a, b in shapes) > 200e9:
            count -= 1
        return dict(kind=kind, qtype=qtype, m=m, count=count,
                    shapes=",".join("%dx%d" % s for s in shapes), x=x, y=_one(rng, "f32", "bf16"))
    return dict(kind=kind, qtype=qtype, n=_log(rng, 300, 16384), k=_mult(_log(rng, 256, 4096), kq))


# ---------------------------------------------------------------------------
# inputs: weights ~ N(0, 0.02), activations ~ N(0, 1), norm weights about 1
# ---------------------------------------------------------------------------

class _Draws:
    """The tensors of one seed, drawn on the GPU in a fixed order."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 1000003 + 17)

    def normal(self, *shape, std=1.0, mean=0.0):
        t = torch.randn(*shape, generator=self.g, device=DEV, dtype=torch.float32)
        if std != 1.0:
            t.mul_(std)
        return t.add_(mean) if mean else t

    def weights(self, n, k):
        return self.normal(n, k, std=0.02)

    def acts(self, m, k, dtype):
        return self.normal(m, k).to(dtype)


def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split(",")]


def _draw_inputs(case, seed, weight):
    """Inputs of a case; each fp32 weight matrix goes through `weight`."""
    g, x = _Draws(seed), DTYPES.get(case.get("x"))
    if case["kind"] == "load":
        return dict(w=g.weights(case["n"], case["k"]))
    if case["kind"] == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        s = dict(w=weight(g.weights(n, k)))
        s["x"] = g.normal(m, k) if case["pro"] else g.acts(m, k, x)
        s["gamma"] = g.normal(k, std=0.1, mean=1.0) if case["pro"] else None
        s["residual"] = g.normal(m, n).to(DTYPES[case["y"]]) if case["epi"] == "add" else None
        return s
    if case["kind"] == "chain":
        m, d, ff, nqkv = case["m"], case["d"], case["ff"], case["nqkv"]
        s = dict(h=g.normal(m, d), layers=[])
        for _ in range(case["layers"]):
            s["layers"].append(dict(
                qkv=weight(g.weights(nqkv, d)), o=weight(g.weights(d, d)),
                gate_up=weight(g.weights(2 * ff, d)), down=weight(g.weights(d, ff)),
                attn=g.acts(m, d, x), g1=g.normal(d, std=0.1, mean=1.0),
                g2=g.normal(d, std=0.1, mean=1.0)))
        return s
    return dict(layers=[(weight(g.weights(n, k)), g.acts(case["m"], k, x))
                        for _ in range(case["count"]) for k, n in _shapes(case)])


def prepare(case, seed):
    """Quantized weights and activations on the GPU; for stacks also the op
    array and the outputs that a program keeps from step to step."""
    # A cached stack plan keeps tables in its op array's workspace.  Plans of
    # op arrays that are gone are dropped before their memory is used again, as
    # eb_qlinear_stack requires of a program that replaces its models.
    eb.stack_cache_clear()
    s = _draw_inputs(case, seed, lambda w: eb.quantize(w, case["qtype"]))
    s["case"] = case
    if case["kind"] == "chain":
        m, xdt = case["m"], DTYPES[case["x"]]
        h = torch.empty_like(s["h"])
        act = torch.empty(m, case["ff"], dtype=xdt, device=DEV)
        entries, qkvs = [], []
        for L in s["layers"]:
            qkv = torch.empty(m, case["nqkv"], dtype=xdt, device=DEV)
            norm = dict(x_dtype=xdt, prologue="rmsnorm", eps=EPS)
            entries += [
                (L["qkv"], h, qkv, dict(norm, norm_weight=L["g1"])),
                (L["o"], L["attn"], h, dict(epilogue="add", residual=h)),
                (L["gate_up"], h, act, dict(norm, norm_weight=L["g2"], epilogue="glu")),
                (L["down"], act, h, dict(epilogue="add", residual=h)),
            ]
            qkvs.append(qkv)
        s.update(out=dict(h=h, act=act, qkv=qkvs), ops=eb.make_ops(entries))
    elif case["kind"] == "layers":
        ydt = DTYPES[case["y"]]
        m, per = case["m"], len(_shapes(case))
        outs, ys = [], [None] * len(s["layers"])
        for j, (_, n) in enumerate(_shapes(case)):
            # outputs of one shape side by side where each then starts on 16 bytes
            if m * n * ydt.itemsize % 16 == 0:
                outs.append(torch.empty(case["count"], m, n, dtype=ydt, device=DEV))
                ys[j::per] = list(outs[-1])
            else:
                ys[j::per] = [torch.empty(m, n, dtype=ydt, device=DEV) for _ in range(case["count"])]
                outs += ys[j::per]
        s.update(ops=eb.make_ops([(w, x, y) for (w, x), y in zip(s["layers"], ys)]), out=outs)
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "linear":
        return eb.qlinear_fused(
            state["w"], state["x"], out_dtype=DTYPES[case["y"]], x_dtype=DTYPES[case["x"]],
            prologue=case["pro"] or None, norm_weight=state["gamma"], eps=EPS if case["pro"] else 0.0,
            epilogue=case["epi"] or None, residual=state["residual"], path=case["path"])
    if case["kind"] == "load":
        qw = eb.quantize(state["w"], case["qtype"])
        blocks = eb.to_canonical(qw)
        back = eb.from_canonical(blocks, case["qtype"], case["n"], case["k"])
        return [qw.buf, blocks, back.buf]
    if case["kind"] == "chain":  # the tokens' embeddings start the residual stream
        state["out"]["h"].copy_(state["h"])
    eb.qlinear_stack(state["ops"])
    return state["out"]


def work(case):
    """Each input read once, each output written once; 2 m n k operations."""
    wb = CODE_BITS[case["qtype"]] / 8
    if case["kind"] == "load":  # fp32 in, blocks out; blocks in, canonical out; and back
        return {"bytes": case["n"] * case["k"] * (4 + 5 * wb), "flops": 0}
    if case["kind"] == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        ys = 4 if case["y"] == "f32" else 2
        nb = n * k * wb + m * k * (4 if case["pro"] else 2) + (4 * k if case["pro"] else 0)
        nb += m * n * ys * (0.5 if case["epi"] == "glu" else 2 if case["epi"] == "add" else 1)
        return {"bytes": nb, "flops": 2 * m * n * k}
    m = case["m"]
    if case["kind"] == "layers":
        ys = 4 if case["y"] == "f32" else 2
        nb = sum(n * k * wb + 2 * m * k + ys * m * n for k, n in _shapes(case))
        return {"bytes": case["count"] * nb,
                "flops": case["count"] * sum(2 * m * n * k for k, n in _shapes(case))}
    d, ff, nqkv, layers = case["d"], case["ff"], case["nqkv"], case["layers"]
    nw = d * nqkv + d * d + 3 * d * ff
    # the stream h in and out once per layer's two updates, attention in, QKV
    # and gated product out, gated product in, norm weights
    nb = nw * wb + m * (4 * 4 * d + 2 * d + 2 * nqkv + 4 * ff) + 8 * d
    return {"bytes": layers * nb, "flops": layers * 2 * m * nw}


def tolerance(case):
    """About four times the error against exact() of the formats' products:
    an output of 16 bits is off by 2.5e-4 (binary16) or 1.7e-3 (bfloat16), and
    so is a product whose weights are rounded once to 16 bits (binary16
    activations off the one-row path; bfloat16 ones above 128 rows); bfloat16
    pairs are 2e-6 off, 32-bit sums of exact products 1e-7.  A gated product
    is off by up to 1.7 times its two factors' error.  In a chain the roundings
    travel: 1.6e-3 after 32 layers in binary16, 3.5e-3 and 8e-3 in bfloat16 at
    50 and 816 rows."""
    if case["kind"] == "load":
        return "exact"
    bf16, large = case["x"] == "bf16", case["m"] > 128
    if case["kind"] == "chain":
        return {"rel": (3e-2 if large else 1.4e-2) if bf16 else 6e-3, "max": 0.3 if bf16 else 0.1}
    rel = {"f32": 0.0, "f16": 2.5e-4, "bf16": 1.7e-3}[case["y"]]
    if case.get("path") == "mfma_i8" or (case["m"] == 1 and not case.get("pro")):
        rel += 1e-6
    elif bf16:
        rel += 1.7e-3 if large else 2.5e-6
    else:
        rel += 2.5e-4
    if case.get("pro"):  # an activation at a tie may round the other way
        rel += 1e-4 if bf16 else 2e-5
    rel *= 4 * (1.7 if case.get("epi") == "glu" else 1.0)
    return {"rel": rel, "max": min(0.9, 20 * rel)}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------

def _away(t):
    return torch.sign(t) * torch.floor(t.abs() + 0.5)


def _half(t):
    return t.to(torch.float32).to(torch.float16).double()


def _div(t, d):
    return torch.where(d == 0, torch.zeros_like(t), t / torch.where(d == 0, torch.ones_like(d), d))


def _signed_max(t):
    return torch.gather(t, -1, t.abs().argmax(-1, keepdim=True))


def _fl32(t):
    return t.to(torch.float32).double()


def _w_hat(w, qtype):
    """w_hat = dequant(quant(W)) of the formats' definitions, in float64."""
    n, k = w.shape
    if qtype == "q6_s":
        b = w.double().view(n, k // 256, 16, 16)
        sub = _fl32(_signed_max(b) / -32.0)
        d = _half(_fl32(sub.abs().amax(2, keepdim=True) / 127.0))
        e = d * _away(_div(sub, d.expand_as(sub))).clamp(-127, 127)
        q = torch.floor(_div(b, e.expand_as(b)) + 0.5).clamp(-32, 31)
        return torch.where(e == 0, torch.zeros_like(q), q * e).view(n, k)
    b = w.double().view(n, k // 32, 32)
    if qtype == "q8_0":
        d = _half(_fl32(b.abs().amax(-1, keepdim=True) / 127.0))
        return (_away(_div(b, d.expand_as(b))).clamp(-127, 127) * d).view(n, k)
    d = _half(_fl32(_signed_max(b) / -8.0))
    q = torch.floor(_div(b, d.expand_as(b)) + 0.5).clamp(-8, 7)
    return torch.where(d == 0, torch.zeros_like(q), q * d).view(n, k)


def _norm(h, gamma, dtype):
    h = h.double()
    x = h * gamma.double() / torch.sqrt(EPS + (h * h).mean(-1, keepdim=True))
    return x.to(torch.float32).to(dtype).double()


def _glu(y):
    g, u = y[:, 0::2], y[:, 1::2]
    return g / (1.0 + torch.exp(-g)) * u


def _x8(x):
    """Activations as the int8 path takes them: per 32 along k, codes times scale."""
    b = x.double().view(x.shape[0], -1, 32)
    s = _fl32(b.abs().amax(-1, keepdim=True) / 127.0)
    return (_away(_div(b, s.expand_as(b))).clamp(-127, 127) * s).view_as(x)


def exact(case, seed):
    if case["kind"] == "load":
        return None  # whole bytes, compared as they are
    s = _draw_inputs(case, seed, lambda w: w)
    qtype, xdt = case["qtype"], DTYPES[case["x"]]

    def mm(x, w):
        return x.double() @ _w_hat(w, qtype).t()

    if case["kind"] == "linear":
        x = _norm(s["x"], s["gamma"], xdt) if case["pro"] else s["x"]
        y = mm(_x8(x) if case["path"] == "mfma_i8" else x, s["w"])
        if case["epi"] == "add":
            y = y + s["residual"].double()
        return _glu(y) if case["epi"] == "glu" else y
    if case["kind"] == "layers":
        m, per, ys = case["m"], len(_shapes(case)), DTYPES[case["y"]].itemsize
        outs, y = [], [mm(x, w) for w, x in s["layers"]]
        for j, (_, n) in enumerate(_shapes(case)):
            outs += [torch.stack(y[j::per])] if m * n * ys % 16 == 0 else y[j::per]
        return outs
    h, qkvs, act = s["h"].double(), [], None
    for L in s["layers"]:
        qkvs.append(mm(_norm(h, L["g1"], xdt), L["qkv"]))
        h = h + mm(L["attn"], L["o"])
        act = _glu(mm(_norm(h, L["g2"], xdt), L["gate_up"]))
        h = h + mm(act.to(torch.float32).to(xdt), L["down"])
    return dict(h=h, act=act, qkv=qkvs)
