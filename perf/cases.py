"""The work a program has libbifattn do: decode steps over a shared context.

Every case is one decode-attention step of one layer, called as a serving or
sampling program calls it: a plan made once for the layer's shape, the caches
resident in device memory, and per step the query of the new tokens (with an
append of their keys and values where the case says so). Shapes: the layers of
this repository's benchmark, plus the two ends it leaves out (a small odd
batch that appends each step, and grouped heads of 64 dims).

Fields of a case: b samples, h query heads, g KV groups, d head dimension,
m_c context keys, m_d rows of each sample's decode cache, n new tokens per
sample, kv cache element type, ragged (each sample's decode length its own,
else all m_d), append (the step first appends its own keys and values).
"""
import math

import torch

import paper_2403_08845_amd as bif

BITS = {"bf16": 16, "fp8_e4m3": 8, "int8": 8, "int4": 4}
QMAX = {"fp8_e4m3": 448.0, "int8": 127.0, "int4": 7.0}
SIGMAS = 4.5  # code caches: standard deviations at the largest code


def _case(b, h, g, d, m_c, m_d, n=1, kv="bf16", ragged=False, append=False, **name):
    return dict(name, b=b, h=h, g=g, d=d, m_c=m_c, m_d=m_d, n=n, kv=kv, ragged=ragged,
                append=append)


def listed():
    return [
        # a toy layer: latency and launches only
        _case(4, 4, 4, 64, 128, 16, name="tiny_mha_b4_mc128"),
        # 7B-shaped multi-head layers sampling 16 and 32 completions of an 8k prompt
        _case(16, 32, 32, 128, 8192, 256, name="mha7b_b16_mc8k_md256"),
        _case(32, 32, 32, 128, 8192, 512, name="mha7b_b32_mc8k_md512"),
        # a multi-query layer, 128 completions of a 16k prompt
        _case(128, 32, 1, 128, 16384, 512, name="mqa_b128_mc16k_md512"),
        # a grouped layer, 256 completions of a 32k prompt that end at different lengths
        _case(256, 32, 8, 128, 32768, 1024, ragged=True, name="gqa8_b256_mc32k_ragged1024"),
        # four draft tokens per sample verified in one step
        _case(32, 32, 32, 128, 8192, 512, n=4, name="mha7b_b32_mc8k_md512_draft4"),
        # quantized caches
        _case(32, 32, 32, 128, 8192, 512, kv="fp8_e4m3", name="mha7b_b32_mc8k_md512_fp8"),
        _case(32, 32, 32, 128, 8192, 512, kv="int8", name="mha7b_b32_mc8k_md512_int8"),
        _case(32, 32, 32, 128, 8192, 512, kv="int4", name="mha7b_b32_mc8k_md512_int4"),
        _case(128, 32, 1, 128, 16384, 512, kv="fp8_e4m3", name="mqa_b128_mc16k_md512_fp8"),
        # one generation step of a small odd batch: append, then attend
        _case(5, 32, 8, 128, 3001, 200, ragged=True, append=True, name="gqa8_b5_mc3001_step"),
        # grouped heads of 64 dims, odd context, ragged
        _case(64, 16, 4, 64, 4097, 384, ragged=True, name="gqa4_d64_b64_mc4097_ragged384"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A layer between the listed ones: any head grouping, size, cache type
    and mode of theirs, no dearer than the largest."""
    limit = _cost(max(listed(), key=_cost))
    while True:
        kind = rng.choice(("mha", "mha", "gqa", "gqa", "mqa"))
        h = rng.choice((4, 8, 16, 24, 32, 32, 40))
        g = h if kind == "mha" else 1 if kind == "mqa" else rng.choice(
            [x for x in (2, 4, 8) if h % x == 0 and x < h])
        d = rng.choice((64, 128, 128, 128))
        c = _case(b=_log_int(rng, 2, 256 if kind != "mha" else 48), h=h, g=g, d=d,
                  m_c=_log_int(rng, 128, 32768), m_d=_log_int(rng, 8, 1024),
                  n=rng.choice((1, 1, 1, 2, 4)),
                  kv=rng.choice(("bf16", "bf16", "bf16", "fp8_e4m3", "int8", "int4")),
                  ragged=rng.random() < 0.5, append=rng.random() < 0.25)
        if h // g * c["n"] <= 64 and _cost(c) <= limit:
            return c


def _mean_len(c):
    """Mean decode length: uniform in [n, m_d] when ragged."""
    return (c["n"] + c["m_d"]) / 2 if c["ragged"] else c["m_d"]


def work(case):
    """One copy of the context, every sample's valid decode rows and q read
    once, the outputs written once; the products of q and K and of the
    weights and V."""
    c = case
    rows = c["m_c"] + c["b"] * _mean_len(c)
    row = c["d"] * BITS[c["kv"]] / 8
    q = c["b"] * c["h"] * c["n"] * c["d"]
    new = 4 * c["b"] * c["g"] * c["n"] * row if c["append"] else 0  # read and written, K and V
    keys = c["m_c"] + _mean_len(c) - (c["n"] - 1) / 2
    return {"bytes": 2 * c["g"] * row * rows + q * (2 + 4) + new, "flops": 4 * q * keys}


def _cost(c):
    w = work(c)
    return max(w["bytes"] / 5e12, w["flops"] / 1e15)


def _cache(c, gen, *rows):
    """Unit normal cache rows of the case's element type; int4 codes packed
    two to a byte, the even one in the low nibble."""
    d = c["d"]
    x = torch.randn(*rows, d, generator=gen, device="cuda", dtype=torch.bfloat16)
    if c["kv"] == "bf16":
        return x
    top = QMAX[c["kv"]]
    out = torch.empty(*rows, d // 2 if c["kv"] == "int4" else d, dtype=torch.uint8, device="cuda")
    for part, dst in zip(x.view(-1, rows[-1], d).split(256), out.view(-1, rows[-1], out.shape[-1]).split(256)):
        y = (part.float() * (top / SIGMAS)).clamp_(-top, top)
        if c["kv"] == "fp8_e4m3":
            dst.copy_(y.to(torch.float8_e4m3fn).view(torch.uint8))
        elif c["kv"] == "int8":
            dst.copy_(y.round_().to(torch.int8).view(torch.uint8))
        else:
            k = y.round_().to(torch.int16) & 15
            dst.copy_((k[..., 0::2] | (k[..., 1::2] << 4)).to(torch.uint8))
    return out


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    b, h, g, d, n = (c[k] for k in ("b", "h", "g", "d", "n"))
    x = {"q": torch.randn(b, h, n, d, generator=gen, device="cuda", dtype=torch.bfloat16),
         "Kc": _cache(c, gen, g, c["m_c"]), "Vc": _cache(c, gen, g, c["m_c"]),
         "Kd": _cache(c, gen, b, g, c["m_d"]), "Vd": _cache(c, gen, b, g, c["m_d"])}
    if c["ragged"]:
        x["lens"] = torch.randint(n, c["m_d"] + 1, (b,), generator=gen, device="cuda",
                                  dtype=torch.int32)
    else:
        x["lens"] = torch.full((b,), c["m_d"], dtype=torch.int32, device="cuda")
    if c["append"]:
        x["k_new"], x["v_new"] = _cache(c, gen, b, g, n), _cache(c, gen, b, g, n)
    x["k_scale"] = x["v_scale"] = None
    if c["kv"] != "bf16":  # per-group scales: groups differ by up to 2x either way
        for k in ("k_scale", "v_scale"):
            u = torch.rand(g, generator=gen, device="cuda")
            x[k] = torch.exp2(2 * u - 1) * (SIGMAS / QMAX[c["kv"]])
    return x


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    x["append"] = c["append"]
    x["plan"] = bif.Plan(c["b"], c["h"], c["g"], c["d"], c["m_c"], c["m_d"], n=c["n"], kv=c["kv"])
    x["out"] = torch.empty(c["b"], c["h"], c["n"], c["d"], dtype=torch.float32, device="cuda")
    if c["append"]:  # the step's own rows are the last of the valid ones afterwards
        x["before"] = x["lens"] - c["n"]
    return x


def run(state):
    s = state
    if s["append"]:
        # the program's own record of the lengths goes to the device, then the
        # step's rows are appended (rows of a rejected step are written over)
        s["lens"].copy_(s["before"])
        bif.bifattn_append_kv(s["plan"], s["k_new"], s["v_new"], s["Kd"], s["Vd"], s["lens"])
    if s["k_scale"] is None:
        bif.bifattn_decode(s["plan"], s["q"], s["Kc"], s["Vc"], s["Kd"], s["Vd"], s["lens"],
                           s["out"])
    else:
        bif.bifattn_decode_scaled(s["plan"], s["q"], s["Kc"], s["Vc"], s["Kd"], s["Vd"],
                                  s["lens"], s["k_scale"], s["v_scale"], s["out"])
    if s["append"]:
        return {"out": s["out"], "Kd": s["Kd"], "Vd": s["Vd"], "lens": s["lens"]}
    return {"out": s["out"]}


def tolerance(case):
    """The softmax weights enter the value products rounded to bf16: measured
    1.1e-3 to 1.7e-3 of the outputs' norm against 64 bits, and single values
    up to 1.0e-2 of the outputs' root mean square off with bf16 caches and
    2.0e-2 with code caches, whose groups differ in scale."""
    return {"rel": 6e-3, "max": 8e-2}


def _values(t, c, scale):
    """A cache tensor [..., g, rows, d] as float64 values."""
    if c["kv"] == "bf16":
        return t.double()
    if c["kv"] == "fp8_e4m3":
        v = t.view(torch.float8_e4m3fn).double()
    elif c["kv"] == "int8":
        v = t.view(torch.int8).double()
    else:
        k = torch.stack((t & 15, t >> 4), -1).flatten(-2).to(torch.int16)
        v = (k - 16 * (k > 7)).double()
    return v * scale.double().view(-1, 1, 1)


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    b, h, g, d, n, m_c, m_d = (c[k] for k in ("b", "h", "g", "d", "n", "m_c", "m_d"))
    p = h // g
    if c["append"]:
        for dst, src in ((x["Kd"], x["k_new"]), (x["Vd"], x["v_new"])):
            for i, end in enumerate(x["lens"].tolist()):
                dst[i, :, end - n:end] = src[i]
    q = x["q"].double().view(b, g, p * n, d) / math.sqrt(d)
    out = torch.empty(b, g, p * n, d, dtype=torch.float64, device="cuda")
    ks, vs = (x[k] if x[k] is not None else torch.ones(g, device="cuda")
              for k in ("k_scale", "v_scale"))
    pos = torch.arange(m_d, device="cuda")
    token = torch.arange(p * n, device="cuda") % n
    for j in range(g):  # group by group: the context's part, then each sample's own
        kc = _values(x["Kc"][j:j + 1], c, ks[j:j + 1])[0]
        vc = _values(x["Vc"][j:j + 1], c, vs[j:j + 1])[0]
        for i0 in range(0, b, 32):
            i1 = min(b, i0 + 32)
            qj = q[i0:i1, j].contiguous()
            kd = _values(x["Kd"][i0:i1, j:j + 1], c, ks[j:j + 1])[:, 0]
            vd = _values(x["Vd"][i0:i1, j:j + 1], c, vs[j:j + 1])[:, 0]
            sc = (qj.view(-1, d) @ kc.t().contiguous()).view(i1 - i0, p * n, m_c)
            sd = torch.bmm(qj, kd.transpose(1, 2).contiguous())
            # token r of n sees the rows up to and including its own
            seen = pos < (x["lens"][i0:i1, None, None] - (n - 1) + token[None, :, None])
            sd = sd.masked_fill(~seen, -math.inf)
            m = torch.maximum(sc.amax(-1, keepdim=True), sd.amax(-1, keepdim=True))
            sc, sd = (sc - m).exp_(), (sd - m).exp_()
            total = sc.sum(-1, keepdim=True) + sd.sum(-1, keepdim=True)
            acc = (sc.view(-1, m_c) @ vc).view(i1 - i0, p * n, d) + torch.bmm(sd, vd)
            out[i0:i1, j] = acc / total
    out = out.view(b, h, n, d)
    if c["append"]:
        return {"out": out, "Kd": None, "Vd": None, "lens": None}
    return {"out": out}
