"""The performance cases of the BAPS library: what its users call it for.

A case is one call of the fused attention (a prompt, a chunk of a prompt, an
encoder layer, a decode step), of the HiF8 codec (a tensor stored and read
back) or of the standalone softmax-block step.  Sizes follow the library's
five workloads and benchmark (Llama-3-8B-shaped GQA 32/8 at head dimension
128, the encoder's 16 heads at head dimension 64), with short, ragged and
chunked sizes beside them.

listed() holds twelve cases, draw() gives more of the same ranges, prepare()
makes a case's inputs on the GPU, run() is the call, work() its least bytes
and operations, tolerance() what another correct implementation may differ by
and exact() the method in 64 bits.
"""
from __future__ import annotations

import math

import torch

import paper_2602_02071_amd as baps

DEV = "cuda:0"
LOG2E = 1.4426950408889634
MODES = {"e2e": baps.BAPS_MODE_E2E_HIF8, "default": baps.BAPS_MODE_DEFAULT, "exp2": baps.BAPS_MODE_EXP2_HIF8}
CODEC_FLAGS = baps.BAPS_HIF8_SATURATE

# Inputs of the attention cases: "normal" is iid N(0, 1); "outliers" scales 1 %
# of the channels of Q and K by 20 (what LLM activations show); "lognormal"
# gives every cached key its own norm.  sink: the first keys scaled by 8.
ATTENTION = dict(kind="attention", B=1, Hq=32, Hkv=8, Sq=1, Sk=1, D=128, causal=True, block=128, mode="e2e",
                 qk="bf16", out="fp32", dist="normal", sink=0, entry="helper")


def _attention(name=None, **kw):
    c = dict(ATTENTION)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one head of 256 positions, where latency and launches count
        _attention("tiny_256_d64", Hq=1, Hkv=1, Sq=256, Sk=256, D=64, causal=False, block=64),
        # a short prompt of an odd length (chat turns): few query tiles for the chip
        _attention("prompt_509", Sq=509, Sk=509, dist="outliers"),
        # the benchmark's prefill
        _attention("prefill_4096", Sq=4096, Sk=4096, dist="outliers"),
        # chunked prefill: the next 777 tokens of a prompt against 6500 cached keys, bf16 output for the next GEMM
        _attention("chunk_777_of_6500", Sq=777, Sk=6500, block=64, dist="outliers", sink=4, out="bf16"),
        # the largest: a long document in one call
        _attention("prefill_32768", Sq=32768, Sk=32768, dist="outliers", sink=4),
        # encoder layer (ViT / multimodal): batch of 8, head dimension 64, no mask
        _attention("encoder_4096_d64", B=8, Hq=16, Hkv=16, Sq=4096, Sk=4096, D=64, causal=False, block=64),
        # encoder layer on FP8 Q/K at an odd token count (37 x 37 patches)
        _attention("encoder_fp8_1369_d64", B=4, Hq=16, Hkv=16, Sq=1369, Sk=1369, D=64, causal=False, qk="fp8",
                   entry="ex"),
        # batched decode of a serving loop with its own output buffers: streams the KV cache
        _attention("decode_b64_8192", B=64, Sq=1, Sk=8192, causal=False, dist="lognormal", entry="buffers"),
        # one sequence's decode step over a long context, workspace kept by the program
        _attention("decode_b1_32768", Sq=1, Sk=32768, dist="lognormal", entry="split"),
        # speculative decode: 6 draft tokens verified for 4 sequences over an odd context length
        _attention("draft6_b4_3001", B=4, Sq=6, Sk=3001, block=64, dist="lognormal", out="bf16", entry="split"),
        # a tensor stored in HiF8 and read back (ragged length)
        dict(name="codec_100000003", kind="codec", n=100000003),
        # the vector-side step on given scores, the benchmark's shape
        dict(name="softmax_16384x8192", kind="softmax", rows=16384, cols=8192, block=128, masked=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: prompts, chunks and encoder layers of 16 to 12000
    queries, decode steps of 1 to 64 sequences over 300 to 40000 keys, codec
    tensors of 2^12 to 2^27 elements, score matrices of 16 to 16384 rows; at
    most half the work of the largest listed case."""
    most = work(listed()[4])["flops"] / 2
    while True:
        kind = rng.choice(("prompt", "prompt", "chunk", "encoder", "encoder", "decode", "decode", "draft", "codec",
                           "softmax"))
        if kind == "codec":
            return dict(kind="codec", n=_log(rng, 1 << 12, 1 << 27))
        if kind == "softmax":
            c = dict(kind="softmax", rows=_log(rng, 16, 16384), cols=_log(rng, 256, 32768),
                     block=rng.choice((64, 128, 256)), masked=rng.random() < 0.3)
            if rng.random() < 0.7:
                c["cols"] -= c["cols"] % 4              # most programs pad their rows to 16 bytes
            if c["rows"] * c["cols"] <= 1 << 27:
                return c
            continue
        block = rng.choice((64, 128, 128))
        hq, hkv = rng.choice(((32, 8), (32, 8), (8, 2), (16, 16), (8, 8)))
        out = rng.choice(("fp32", "bf16"))
        dist = rng.choice(("normal", "outliers"))
        if kind == "prompt":
            s = _log(rng, 16, 12000)
            c = _attention(B=_log(rng, 1, 8), Hq=hq, Hkv=hkv, Sq=s, Sk=s, block=block, out=out, dist=dist,
                           sink=rng.choice((0, 4)), mode=rng.choice(("e2e",) * 6 + ("default", "exp2")), entry="ex")
        elif kind == "chunk":
            s = _log(rng, 64, 2048)
            c = _attention(B=rng.choice((1, 1, 2)), Hq=hq, Hkv=hkv, Sq=s, Sk=s + _log(rng, 256, 16384), block=block,
                           out=out, dist=dist, sink=rng.choice((0, 4)), entry="ex")
        elif kind == "encoder":
            s = _log(rng, 64, 6000)
            h = rng.choice((8, 12, 16))
            c = _attention(B=_log(rng, 1, 16), Hq=h, Hkv=h, Sq=s, Sk=s, D=rng.choice((64, 64, 128)), causal=False,
                           block=block, out=out, qk=rng.choice(("bf16", "bf16", "fp8")),
                           mode=rng.choice(("e2e",) * 6 + ("default", "exp2")), entry="ex")
        else:
            c = _attention(B=_log(rng, 1, 64), Hq=hq, Hkv=hkv, Sq=1 if kind == "decode" else rng.randint(2, 8),
                           Sk=_log(rng, 300, 40000), block=block, out=out, dist="lognormal",
                           qk=rng.choice(("bf16", "bf16", "fp8")), entry="split")
        w = work(c)
        if w["flops"] <= most and w["bytes"] <= 1.1e9:
            return c


# ------------------------------------------------------------------ the calls
def _make_qkv(c, seed):
    """bf16 q [B,Hq,Sq,D], k, v [B,Hkv,Sk,D] of a case, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)

    q, k, v = (normal(c["B"], h, s, c["D"]) for h, s in ((c["Hq"], c["Sq"]), (c["Hkv"], c["Sk"]), (c["Hkv"], c["Sk"])))
    if c["dist"] == "outliers":
        ch = torch.randperm(c["D"], generator=g, device=DEV)[:math.ceil(0.01 * c["D"])]
        q[..., ch] *= 20.0
        k[..., ch] *= 20.0
    elif c["dist"] == "lognormal":
        k *= torch.exp(0.5 * normal(c["B"], c["Hkv"], c["Sk"], 1))
    if c["sink"]:
        k[:, :, :c["sink"]] *= 8.0
    return q.bfloat16(), k.bfloat16(), v.bfloat16()


def _fp8(x):
    """(E4M3 codes as uint8, power-of-two scale) of a tensor."""
    scale = 2.0 ** math.ceil(math.log2(float(x.abs().max()) / 448.0))
    return (x.float() / scale).to(torch.float8_e4m3fn).view(torch.uint8), scale


def _attention_state(c, seed):
    q, k, v = _make_qkv(c, seed)
    knobs = {}
    if c["mode"] != "e2e":
        knobs["mode"] = MODES[c["mode"]]
    if c["out"] == "bf16":
        knobs["out_bf16"] = True
    if c["qk"] == "fp8":
        (q, qs), (k, ks) = _fp8(q), _fp8(k)
        knobs["qk_scales"] = (qs, ks)
    s = dict(case=c, q=q, k=k, v=v, knobs=knobs)
    shape = (c["B"], c["Hq"], c["Hkv"], c["Sq"], c["Sk"], c["D"])
    if c["entry"] in ("buffers", "split"):
        s["shape"] = shape
        s["o"] = torch.empty(q.shape, dtype=torch.bfloat16 if c["out"] == "bf16" else torch.float32, device=DEV)
        s["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device=DEV)
    if c["entry"] == "split":
        n = baps.baps_attention_split_workspace(*shape, c["block"], **knobs)
        s["workspace"], s["bytes"] = torch.empty(max(n, 1), dtype=torch.uint8, device=DEV), n
    return s


def prepare(case, seed):
    if case["kind"] == "attention":
        return _attention_state(case, seed)
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    if case["kind"] == "codec":
        n = case["n"]
        x = torch.randn(n, generator=g, device=DEV, dtype=torch.float32)
        # activations: most of them ordinary, some far into the tapered range
        x *= torch.exp2(4.0 * torch.randn(n, generator=g, device=DEV, dtype=torch.float32))
        return dict(case=case, x=x, codes=torch.empty(n, dtype=torch.uint8, device=DEV),
                    y=torch.empty(n, dtype=torch.float32, device=DEV))
    rows, cols, block = case["rows"], case["cols"], case["block"]
    nblk = -(-cols // block)
    s = 4.0 * torch.randn((rows, cols), generator=g, device=DEV, dtype=torch.float32)
    if case["masked"]:                                  # the upper triangle of a square causal tile, at the last columns
        keep = cols - torch.arange(rows, device=DEV) % max(1, cols // 2)
        s.masked_fill_(torch.arange(cols, device=DEV)[None, :] >= keep[:, None], float("-inf"))
    return dict(case=case, s=s, codes=torch.empty((rows, cols), dtype=torch.uint8, device=DEV),
                shift=torch.empty((rows, nblk), dtype=torch.int32, device=DEV),
                m=torch.empty(rows, dtype=torch.float32, device=DEV),
                d=torch.empty(rows, dtype=torch.float32, device=DEV),
                restarted=torch.empty((rows, nblk), dtype=torch.uint8, device=DEV))


def run(state):
    c = state["case"]
    if c["kind"] == "codec":
        baps.hif8_encode(state["x"], state["codes"], c["n"], CODEC_FLAGS)
        baps.hif8_decode(state["codes"], state["y"], c["n"])
        return dict(codes=state["codes"], y=state["y"])
    if c["kind"] == "softmax":
        baps.baps_softmax_block(state["s"], c["rows"], c["cols"], c["cols"], c["block"], 1, 1, 0, state["codes"],
                                state["shift"], state["m"], state["d"], state["restarted"])
        return {k: state[k] for k in ("codes", "shift", "m", "d", "restarted")}
    q, k, v = state["q"], state["k"], state["v"]
    if c["entry"] == "buffers":
        baps.baps_attention_fwd(q, k, v, state["o"], state["lse"], *state["shape"], c["causal"], c["block"])
        return dict(o=state["o"], lse=state["lse"])
    if c["entry"] == "split":
        baps.baps_attention_fwd_split(q, k, v, state["o"], state["lse"], *state["shape"], c["causal"], c["block"],
                                      state["workspace"], state["bytes"], **state["knobs"])
        return dict(o=state["o"], lse=state["lse"])
    o, lse = baps.attention(q, k, v, c["causal"], c["block"], **state["knobs"])
    return dict(o=o, lse=lse)


# ------------------------------------------------------------ work, tolerance
def _pairs(c):
    if not c["causal"]:
        return c["Sq"] * c["Sk"]
    off = c["Sk"] - c["Sq"]                             # bottom-right aligned; Sk >= Sq in every case here
    return c["Sq"] * (off + 1) + c["Sq"] * (c["Sq"] - 1) // 2


def work(case):
    if case["kind"] == "codec":                         # 4 B in + 1 B out, then 1 B in + 4 B out
        return {"bytes": 10 * case["n"], "flops": 0}
    if case["kind"] == "softmax":
        nblk = -(-case["cols"] // case["block"])
        return {"bytes": case["rows"] * (5 * case["cols"] + 5 * nblk + 8), "flops": 0}
    qk_b = 1 if case["qk"] == "fp8" else 2
    o_b = 2 if case["out"] == "bf16" else 4
    q_n = case["B"] * case["Hq"] * case["Sq"]
    k_n = case["B"] * case["Hkv"] * case["Sk"]
    return {"bytes": q_n * (case["D"] * (qk_b + o_b) + 4) + k_n * case["D"] * (qk_b + 2),
            "flops": 4 * case["D"] * _pairs(case) * case["B"] * case["Hq"]}


def tolerance(case):
    """Codes, references and flags are whole values and stay the same.  In the
    attention cases a dot product summed in another order can move a score
    across a rounding boundary of the 8-bit format, which moves one P of the
    row by up to 1/8: rare, largest where outlier channels let few keys carry
    a row (and with the scores' magnitude)."""
    if case["kind"] == "codec":
        return "exact"
    if case["kind"] == "softmax":
        return {"rel": 5e-6, "max": 5e-5, "differ": 0.0}   # d: an fp32 sum of a row
    rel, most = (8e-4, 0.5) if case["dist"] == "outliers" else (6e-4, 0.3)
    if case["qk"] == "fp8":                             # the FP8 matrix instructions keep fewer bits of a sum
        rel = 6e-3
    if case["out"] == "bf16" or case["mode"] == "default":
        rel = 8e-3
    return {"rel": rel, "max": most}


# ------------------------------------------------------------- the 64-bit form
def _hif8(x):
    """HiF8 rounding (ties away from zero, saturating) of finite or -inf values in 64 bits."""
    a = x.abs()
    e = torch.frexp(a).exponent - 1                     # a = 2^e * [1, 2)
    ae = e.abs()
    w = torch.where(ae <= 3, 3, torch.where(ae <= 7, 2, 1))
    w = torch.where(e < -15, 0, w)
    e = torch.maximum(e, torch.full_like(e, -22))       # below 2^-22 the nearest values are 0 and 2^-22
    step = torch.ldexp(torch.ones((), dtype=torch.float64, device=x.device), e - w)
    r = torch.clamp(torch.floor(a / step + 0.5) * step, max=32768.0)
    r = torch.where(a < 2.0 ** -23, torch.zeros_like(r), torch.where(a < 2.0 ** -22, torch.full_like(r, 2.0 ** -22), r))
    return torch.where(torch.isinf(x), x, torch.copysign(r, x))


def _references(bmax, n_b0=1, lam=1.0):
    """Alg. 1's per-block references and integer maximum from the block maxima [..., nblk]; also the restarts."""
    ninf = torch.full_like(bmax[..., 0], float("-inf"))
    m, refs, rst = ninf, [], []
    for j in range(bmax.shape[-1]):
        mx = bmax[..., j]
        t = torch.ceil(_hif8(torch.where(torch.isinf(m) | torch.isinf(mx), ninf, mx - m)))
        restart = torch.isinf(m) | (t > lam) if j >= n_b0 else torch.ones_like(m, dtype=torch.bool)
        hi = torch.maximum(m, torch.ceil(mx))
        ref = torch.where(restart, hi, m)
        m = torch.where(restart, hi, m + torch.clamp(t, min=0.0))
        refs.append(ref)
        rst.append(restart)
    return torch.stack(refs, -1), m, torch.stack(rst, -1)


def _exact_rows(c, s, v):
    """O and lse of score rows s [n, rows, keys] (log2 units, -inf masked) over v [n, keys, D], in 64 bits."""
    n, rows, keys = s.shape
    if c["mode"] == "default":
        m = s.amax(-1, keepdim=True)
        p = torch.exp2(s - m)
        d = p.sum(-1)
        return torch.bmm(p, v) / d[..., None], math.log(2.0) * (m[..., 0] + torch.log2(d))
    nblk = -(-keys // c["block"])
    pad = nblk * c["block"] - keys
    if pad:
        s = torch.nn.functional.pad(s, (0, pad), value=float("-inf"))
        v = torch.nn.functional.pad(v, (0, 0, 0, pad))
    s = s.view(n, rows, nblk, c["block"])
    bmax = s.amax(-1)
    if c["mode"] == "exp2":
        # eq. 2: real-valued running maximum, rescale factors rounded to 8 bits
        refs = torch.cummax(bmax, -1).values
        f = _hif8(torch.exp2(_hif8(torch.diff(refs, dim=-1).neg())))
        w = torch.cat((f.flip(-1).cumprod(-1).flip(-1), torch.ones_like(refs[..., :1])), -1)
        last = refs[..., -1]
    else:
        refs, m, _ = _references(bmax)
        refs = torch.cummax(refs, -1).values            # (a block past the mask keeps the last reference)
        last = refs[..., -1]
        w = torch.exp2(refs - last[..., None])
    p = _hif8(torch.exp2(_hif8(s - refs[..., None])))
    p = (p * w[..., None]).view(n, rows, nblk * c["block"])
    d = p.sum(-1)
    return torch.bmm(p, v) / d[..., None], math.log(2.0) * (last + torch.log2(d))


def _exact_attention(c, seed):
    st = _attention_state(dict(c, entry="helper"), seed)
    q, k, v = st["q"], st["k"], st["v"].double()
    base = LOG2E / math.sqrt(c["D"])
    if c["qk"] == "fp8":
        qs, ks = st["knobs"]["qk_scales"]
        q, k = (x.view(torch.float8_e4m3fn).float() for x in (q, k))
        base *= qs * ks
    scale = float(torch.tensor(base, dtype=torch.float64).float())       # the scale is an fp32 number
    q, k = q.double(), k.double()
    B, Hq, Sq, D = q.shape
    Hkv, Sk = k.shape[1], k.shape[2]
    o = torch.empty((B, Hq, Sq, D), dtype=torch.float64, device=DEV)
    lse = torch.empty((B, Hq, Sq), dtype=torch.float64, device=DEV)
    step = max(1, min(Sq, (1 << 27) // (Hq * Sk)))
    for b in range(B):
        kt = k[b].repeat_interleave(Hq // Hkv, 0).transpose(1, 2).contiguous()
        vr = v[b].repeat_interleave(Hq // Hkv, 0)
        for r0 in range(0, Sq, step):
            r1 = min(Sq, r0 + step)
            n = Sk - Sq + r1 if c["causal"] else Sk      # keys that some row of the chunk sees
            s = torch.bmm(q[b, :, r0:r1].contiguous(), kt[:, :, :n].contiguous()) * scale
            if c["causal"]:
                seen = torch.arange(r0, r1, device=DEV) + Sk - Sq
                s.masked_fill_(torch.arange(n, device=DEV)[None, :] > seen[:, None], float("-inf"))
            o[b, :, r0:r1], lse[b, :, r0:r1] = _exact_rows(c, s, vr[:, :n].contiguous())
    return dict(o=o, lse=lse)


def exact(case, seed):
    if case["kind"] == "attention":
        return _exact_attention(case, seed)
    st = prepare(case, seed)
    if case["kind"] == "codec":
        y = torch.cat([_hif8(x.double()) for x in st["x"].split(1 << 24)])
        return dict(codes=None, y=y)
    m, d = [], []
    block, cols = case["block"], case["cols"]
    for s in st["s"].split(max(1, (1 << 26) // cols)):
        s = torch.nn.functional.pad(s.double(), (0, -cols % block), value=float("-inf")).view(len(s), -1, block)
        refs, mf, _ = _references(s.amax(-1))
        refs = torch.cummax(refs, -1).values
        p = _hif8(torch.exp2(_hif8(s - refs[..., None]))).sum(-1)
        m.append(mf)
        d.append((p * torch.exp2(refs - mf[:, None])).sum(-1))
    return dict(codes=None, shift=None, m=torch.cat(m), d=torch.cat(d), restarted=None)
