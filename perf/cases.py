"""The work the framework is measured on, through its public entry points.

Four kinds of pass, each over the sizes, cache formats, head dims, group sizes
and storage options a caller meets:

* ``decode``: one decode step of a batch through every layer of a cache
  (``append_decode_attn_ptr``, the call of a serving loop whose buffers are
  laid out once, as the benchmark issues it);
* ``chunk``: prefill attention of one chunk over the keys already cached;
* ``prompt``: a whole prompt into an empty sequence -- chunk by chunk,
  attention then materialisation in every layer -- and its first decode step;
* ``calib``: the calibration replay of one traced layer.

Lengths, window codebooks and level matrices follow from the case; keys,
values and queries are seeded unit normals rounded to bf16, with two outlier
channels per KV head scaled by 8 where the case says so (the recipe of the
repository's own workloads).
"""
import math
import random

import torch

from paper_2609_02029_amd import hwkv

# Decode passes append a token each: rows a full unit has left for them.
HEADROOM = 16384
PAGE = hwkv.PAGE_TOKENS
DEV = "cuda"


def _decode(name, **kw):
    c = dict(name=name, kind="decode", layers=1, batch=1, d=128, g=4, hkv=8, sinks=4, windows="",
             full=True, lo=1024, hi=1024, fmt="bf16", paged=False, outliers=False, pick=1)
    c.update(kw)
    return c


def _chunk(name, **kw):
    c = dict(name=name, kind="chunk", d=128, g=4, hkv=8, sinks=4, windows="", full=True, p0=0,
             n=512, fmt="bf16", paged=False, outliers=False, pick=1)
    c.update(kw)
    return c


def _prompt(name, **kw):
    c = dict(name=name, kind="prompt", layers=1, d=128, g=4, hkv=8, sinks=4, windows="", full=True,
             n=1024, cut=1024, fmt="bf16", paged=False, outliers=False, pick=1)
    c.update(kw)
    return c


def _calib(name, **kw):
    c = dict(name=name, kind="calib", d=256, g=6, hkv=4, sinks=4, windows="", hist=131072,
             rows=256, fmt="bf16", outliers=False, pick=1)
    c.update(kw)
    return c


def listed():
    return [
        # interactive decoding with short per-head histories: one sequence,
        # the head shape of the smallest workload, sink + recent caches of
        # 260 and 2,048 tokens in 16 layers; launches and latency count
        _decode("decode_short", layers=16, d=64, g=4, hkv=2, windows="256,2044", full=False,
                lo=4000, hi=4000),
        # the headline: one sequence at 112K context through 16 layers,
        # per-head windows {2K, 8K, 32K, full}
        _decode("decode_112k", layers=16, d=256, g=6, hkv=4, windows="2048,8192,32768",
                lo=114688, hi=114688, pick=3),
        # a long-context batch over an fp8 cache: four ragged sequences
        _decode("decode_fp8", layers=8, batch=4, d=128, g=8, hkv=8, windows="1024,4096,16384",
                lo=24000, hi=64000, fmt="fp8", outliers=True),
        # batched serving: 16 ragged sequences of 16K-64K, paged full units
        _decode("decode_batch16", layers=8, batch=16, d=256, g=6, hkv=4,
                windows="1024,4096,16384", lo=16384, hi=65536, paged=True, pick=4),
        # a busy chat server: many short ragged sequences, binary16 cache
        _decode("decode_batch48", layers=4, batch=48, d=128, g=4, hkv=8, windows="512,1500",
                lo=200, hi=6000, fmt="f16", paged=True),
        # a chat prompt of odd length, materialised chunk by chunk, and its
        # first decode step (time to first token)
        _prompt("prompt_3k", layers=2, d=128, g=4, hkv=8, windows="512,1500", n=2901, cut=1024),
        # chunked prefill beside decoding: a small chunk far into a long
        # context, paged full units
        _chunk("chunk_512", d=128, g=4, hkv=8, windows="2048,8192", p0=49152, n=512, paged=True),
        # the last 8K chunk of the 128K prefill workload, KV head h at level h
        _chunk("chunk_8k_at_120k", d=256, g=6, hkv=4, windows="2048,8192,32768", p0=122880,
               n=8192, pick=0),
        # a ragged chunk over an fp8 cache (staged codes)
        _chunk("chunk_fp8", d=256, g=6, hkv=4, windows="1024,4096,16384", p0=30011, n=1999,
               fmt="fp8", outliers=True),
        # small heads, multi-head attention without grouping, binary16 cache
        _chunk("chunk_f16", d=64, g=1, hkv=32, windows="1024,4096", p0=12288, n=4096, fmt="f16"),
        # calibration at full size: 256 rows of a 128K trace
        _calib("calib_128k", windows="2048,8192,32768"),
        # calibration of a short fp8 trace, ragged sizes
        _calib("calib_fp8", d=128, g=4, hkv=8, windows="250,1024,4096", hist=20011, rows=101,
               fmt="fp8", outliers=True),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _windows(rng, top, least=0):
    n = rng.randint(least, 3)
    return ",".join(str(w) for w in sorted({_logint(rng, 64, max(65, top)) for _ in range(n)}))


def draw(rng):
    """One more case: the kinds alternate at random, sizes over the whole
    range of the listed ones."""
    kind = rng.choice(["decode", "decode", "decode", "chunk", "chunk", "prompt", "calib"])
    while True:
        c = dict(kind=kind, d=rng.choice([64, 128, 128, 256]), g=rng.choice([1, 2, 4, 6, 8]),
                 hkv=rng.randint(1, 8), sinks=rng.choice([0, 1, 4, 4, 16]),
                 fmt=rng.choice(["bf16", "bf16", "f16", "fp8"]), outliers=rng.random() < 0.3,
                 pick=rng.randint(1, 1 << 20))
        if kind == "decode":
            hi = _logint(rng, 300, 120000)
            c.update(layers=rng.randint(4, 16), batch=_logint(rng, 1, 64), lo=max(1, hi // rng.randint(1, 8)),
                     hi=hi, paged=rng.random() < 0.5, full=rng.random() < 0.7,
                     windows=_windows(rng, hi))
        elif kind == "chunk":
            c.update(p0=rng.choice([0, _logint(rng, 100, 120000), _logint(rng, 100, 120000)]),
                     n=_logint(rng, 16, 8192), paged=rng.random() < 0.5, full=rng.random() < 0.7)
            c["windows"] = _windows(rng, c["p0"] + c["n"])
        elif kind == "prompt":
            c.update(layers=rng.randint(1, 4), n=_logint(rng, 200, 8000), cut=rng.choice([512, 1000, 2048]),
                     paged=rng.random() < 0.5, full=rng.random() < 0.7)
            c["windows"] = _windows(rng, c["n"])
        else:
            c["fmt"] = rng.choice(["bf16", "fp8"])
            c.update(hist=_logint(rng, 4096, 131072), rows=_logint(rng, 16, 256))
            c["windows"] = _windows(rng, c["hist"], 1)
        if kind != "calib" and not c["full"] and not c["windows"]:
            c["full"] = True
        w = work(c)
        most = {"decode": (6.0e9, 4e11), "chunk": (4e9, 6.6e12), "prompt": (4e9, 2e12),
                "calib": (2e9, 1e12)}[kind]
        if w["bytes"] <= most[0] and w["flops"] <= most[1] and (kind != "decode" or w["bytes"] >= 2e6):
            return c


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------
def _layers(c):
    return c.get("layers", 1)


def _codebook(c):
    w = [int(x) for x in c["windows"].split(",") if x]
    return w + [0] if c.get("full", True) or not w else w


def _levels(c):
    """[layers][hkv] level indices: head h at level h (pick 0), else drawn
    evenly, with a full unit somewhere if the codebook has one."""
    k = len(_codebook(c))
    if not c["pick"]:
        return [[h % k for h in range(c["hkv"])] for _ in range(_layers(c))]
    r = random.Random(c["pick"])
    flat = [i % k for i in range(_layers(c) * c["hkv"])]
    r.shuffle(flat)
    return [flat[i * c["hkv"]:(i + 1) * c["hkv"]] for i in range(_layers(c))]


def _lengths(c):
    r = random.Random(c["pick"] + 17)
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["batch"])]


def _max_ctx(c):
    if c["kind"] == "decode":
        return c["hi"] + HEADROOM
    if c["kind"] == "chunk":
        return c["p0"] + c["n"] + 512
    return c["n"] + 256 if c["kind"] == "prompt" else c["hist"]


def _held(c, w, n):
    """Positions a unit of window w (0 = full) holds at length n."""
    return n if w == 0 or c["sinks"] + w >= _max_ctx(c) else min(n, c["sinks"] + w)


def _pairs(c, w, p0, n):
    """(query token, visible key) pairs of tokens [p0, p0 + n) under window w."""
    return sum(_held(c, w, t + 1) for t in range(p0, p0 + n))


def _elem(c):
    return 1 if c["fmt"] == "fp8" else 2


def work(c):
    d, g, hkv, e = c["d"], c["g"], c["hkv"], _elem(c)
    cb, lv = _codebook(c), _levels(c)
    if c["kind"] == "decode":
        rows = sum(_held(c, cb[k], n + 1) for row in lv for k in row for n in _lengths(c))
        per = len(lv) * c["batch"] * hkv
        return {"bytes": rows * d * 2.0 * e + per * d * (2 * g + 4 + 4 * g),
                "flops": rows * g * d * 4.0}
    if c["kind"] == "chunk":
        p0, n = c["p0"], c["n"]
        keys = sum(min(p0, _held(c, cb[k], p0 + 1)) for k in lv[0])
        return {"bytes": keys * d * 2.0 * e + n * hkv * d * (4.0 + 6.0 * g),
                "flops": 4.0 * d * g * sum(_pairs(c, cb[k], p0, n) for k in lv[0])}
    if c["kind"] == "prompt":
        n = c["n"]
        rows = sum(_held(c, cb[k], n + 1) for row in lv for k in row)
        return {"bytes": rows * d * 2.0 * e + len(lv) * (n + 1) * hkv * d * (4.0 + 6.0 * g),
                "flops": 4.0 * d * g * sum(_pairs(c, cb[k], 0, n + 1) for row in lv for k in row)}
    rows = _rows(c)
    ws = [int(x) for x in c["windows"].split(",")]
    # one pass over each row's history serves the nested candidates
    return {"bytes": c["hist"] * hkv * d * 4.0 + len(rows) * hkv * g * d * (2.0 + 4.0 * (len(ws) + 1)),
            "flops": 4.0 * d * g * hkv * sum(t + 1 for t in rows)}


def _rows(c):
    r = random.Random(c["pick"] + 5)
    return sorted(r.sample(range(c["hist"] - c["hist"] // 4, c["hist"]), c["rows"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Inputs:
    """Seeded inputs, drawn in a fixed order."""

    def __init__(self, c, seed):
        self.c = c
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed((int(seed) * 1000003 + 12345) % (1 << 62))
        r = random.Random(c["pick"] + 29)
        self.loud = [r.sample(range(c["d"]), 2) for _ in range(c["hkv"])] if c["outliers"] else None

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device=DEV).to(torch.bfloat16)

    def kv(self, n):
        """K and V of n tokens (or sequences): [n, hkv, d]."""
        out = []
        for _ in range(2):
            x = torch.randn((n, self.c["hkv"], self.c["d"]), generator=self.gen, device=DEV)
            if self.loud:
                for h, chans in enumerate(self.loud):
                    for ch in chans:
                        x[:, h, ch] *= 8.0
            out.append(x.to(torch.bfloat16))
        return out

    def q(self, n):
        return self.normal(n, self.c["hkv"] * self.c["g"], self.c["d"])


def _scales(c):
    """fp8 scales: eight standard deviations of the loudest channel reach 448."""
    if c["fmt"] != "fp8":
        return {}
    s = 8.0 * (8.0 if c["outliers"] else 1.0) / 448.0
    return dict(k_scale=s, v_scale=s)


def _cache(c, batch):
    pol = hwkv.policy_set(_layers(c), c["hkv"], c["hkv"] * c["g"], c["d"], c["sinks"], _codebook(c), _levels(c))
    top = _max_ctx(c)
    pages = None
    if c["paged"]:
        cb = _codebook(c)
        full = sum(1 for row in _levels(c) for k in row if _held(c, cb[k], top) == top)
        ends = [n + HEADROOM for n in _lengths(c)] if c["kind"] == "decode" else [top]
        pages = full * sum(-(-n // PAGE) for n in ends)
    return hwkv.cache_alloc(pol, batch, top, kv_format=c["fmt"], n_pages=pages, **_scales(c))


def prepare(c, seed):
    x = _Inputs(c, seed)
    s = {"c": c, "scale": 1.0 / math.sqrt(c["d"])}
    if c["kind"] == "decode":
        s["cache"] = cache = _cache(c, c["batch"])
        for l in range(_layers(c)):
            for b, n in enumerate(_lengths(c)):
                hwkv.prefill_write(cache, l, b, 0, *x.kv(n))
        s["steps"] = [(*x.kv(c["batch"]), x.q(c["batch"])) for _ in range(_layers(c))]
        s["out"] = torch.empty((_layers(c), c["batch"], c["hkv"] * c["g"], c["d"]), device=DEV)
        s["ws"] = torch.empty(max(1, hwkv.decode_workspace_bytes(cache)), dtype=torch.uint8, device=DEV)
        # the addresses a step loop hands over, as the benchmark's does
        s["calls"] = [(l, k.data_ptr(), v.data_ptr(), q.data_ptr(), s["scale"], s["out"][l].data_ptr(),
                       s["ws"].data_ptr(), s["ws"].numel()) for l, (k, v, q) in enumerate(s["steps"])]
    elif c["kind"] == "chunk":
        s["cache"] = cache = _cache(c, 1)
        if c["p0"]:
            hwkv.prefill_write(cache, 0, 0, 0, *x.kv(c["p0"]))
        s["k"], s["v"] = x.kv(c["n"])
        s["q"] = x.q(c["n"])
        s["out"] = torch.empty(s["q"].shape, device=DEV)
        s["ws"] = _prefill_ws(cache, c["n"])
    elif c["kind"] == "prompt":
        s["cache"] = cache = _cache(c, 1)
        s["tokens"] = [(*x.kv(c["n"] + 1), x.q(c["n"] + 1)) for _ in range(_layers(c))]
        s["out"] = torch.empty((_layers(c), c["n"] + 1, c["hkv"] * c["g"], c["d"]), device=DEV)
        s["ws"] = _prefill_ws(cache, min(c["n"], c["cut"]))
        s["dws"] = torch.empty(max(1, hwkv.decode_workspace_bytes(cache)), dtype=torch.uint8, device=DEV)
    else:
        s["k"], s["v"] = x.kv(c["hist"])
        s["q"] = x.q(c["rows"])
        s["rows"] = _rows(c)
        s["windows"] = [int(w) for w in c["windows"].split(",")]
        K, hq = len(s["windows"]), c["hkv"] * c["g"]
        s["outs"] = torch.empty((K + 1, c["rows"], hq, c["d"]), device=DEV)
        s["scores"] = torch.empty((K, c["rows"], hq), device=DEV)
        s["means"] = torch.empty((K, c["hkv"]), device=DEV)
        s["ws"] = torch.empty(hwkv.calib_workspace_bytes(hq, c["d"], c["sinks"], c["hist"], c["rows"],
                                                         n_kv_heads=c["hkv"], kv_format=c["fmt"]),
                              dtype=torch.uint8, device=DEV)
    return s


def _prefill_ws(cache, n):
    need = hwkv.prefill_attn_workspace_bytes(cache, n)
    return torch.empty(need, dtype=torch.uint8, device=DEV) if need else None


def run(s):
    c = s["c"]
    if c["kind"] == "decode":
        stream = torch.cuda.current_stream().cuda_stream
        for layer, k, v, q, scale, out, ws, n in s["calls"]:
            hwkv.append_decode_attn_ptr(s["cache"], layer, k, v, q, scale, out, ws, n, stream)
        return s["out"]
    if c["kind"] == "chunk":
        hwkv.prefill_attn(s["cache"], 0, 0, c["p0"], s["q"], s["k"], s["v"], s["scale"], s["out"], ws=s["ws"])
        return s["out"]
    if c["kind"] == "prompt":
        cache, n = s["cache"], c["n"]
        hwkv.cache_reset_seq(cache, 0)
        for p0 in range(0, n, c["cut"]):
            p1 = min(n, p0 + c["cut"])
            for l, (k, v, q) in enumerate(s["tokens"]):
                hwkv.prefill_attn(cache, l, 0, p0, q[p0:p1], k[p0:p1], v[p0:p1], s["scale"], s["out"][l, p0:p1],
                                  ws=s["ws"])
                hwkv.prefill_write(cache, l, 0, p0, k[p0:p1], v[p0:p1])
        for l, (k, v, q) in enumerate(s["tokens"]):
            hwkv.append_decode_attn(cache, l, k[n:], v[n:], q[n:], s["scale"], s["out"][l, n:], s["dws"])
        return s["out"]
    hwkv.calib_replay(s["k"], s["v"], s["rows"], s["q"], s["windows"], c["sinks"], s["scale"], s["outs"],
                      s["scores"], s["means"], s["ws"], kv_format=c["fmt"], **_scales(c))
    return {"outs": s["outs"], "scores": s["scores"], "means": s["means"]}


def tolerance(c):
    """About four times the error measured against 64 bits.  Decode: fp32
    sums and weights (at most 2.8e-7); over fp8 codes the weights enter the
    value product as two bf16 terms (2.3e-6).  Prefill and the replay round
    each weight to the 16-bit type of the value product: 1.7e-3 with bf16
    (fp8 codes are staged as bf16), 2.1e-4 with binary16.  A prompt's decode
    step is held to its prefill's tolerance."""
    if c["kind"] == "decode":
        return {"rel": 1e-5 if c["fmt"] == "fp8" else 1.5e-6}
    return {"rel": 1e-3 if c["fmt"] == "f16" else 7e-3}


# ---------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _stored(c, x):
    """Values a cache of the case's format holds for bf16 x, in fp64."""
    if c["fmt"] == "f16":
        return x.to(torch.float16).double()
    if c["fmt"] == "fp8":
        s = torch.tensor(_scales(c)["k_scale"], dtype=torch.float32, device=x.device)
        y = (x.float() / s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
        return y.double() * s.double()
    return x.double()


def _attend(q, k, v, pos, window, sinks, scale):
    """q [m, d] at positions pos [m] (ascending) over k, v [n, d] (fp64)."""
    out = torch.empty_like(q)
    step = max(64, min(q.shape[0], (1 << 27) // max(1, k.shape[0])))
    for i in range(0, q.shape[0], step):
        p = pos[i:i + step]
        hi = int(p[-1]) + 1
        lo = max(0, int(p[0]) + 1 - window) if window else 0
        if lo > sinks:
            at = torch.cat([torch.arange(sinks, device=q.device), torch.arange(lo, hi, device=q.device)])
        else:
            at = torch.arange(hi, device=q.device)
        z = (q[i:i + step] @ k[at].T) * scale
        seen = at[None, :] <= p[:, None]
        if window:
            seen &= (at[None, :] < sinks) | (at[None, :] > p[:, None] - window)
        z.masked_fill_(~seen, -math.inf)
        out[i:i + step] = torch.softmax(z, dim=1) @ v[at]
    return out


def _attend_heads(c, out, q, k, v, p0, windows, scale):
    """out, q [n, hq, d] of positions p0.. over k, v [>= p0 + n, hkv, d]."""
    n, d, g = q.shape[0], c["d"], c["g"]
    pos = (p0 + torch.arange(n, device=q.device)).repeat_interleave(g)
    for h in range(c["hkv"]):
        qh = q[:, h * g:(h + 1) * g].reshape(n * g, d).double()
        o = _attend(qh, _stored(c, k[:, h]), _stored(c, v[:, h]), pos, windows[h], c["sinks"], scale)
        out[:, h * g:(h + 1) * g] = o.reshape(n, g, d)


def exact(c, seed):
    x = _Inputs(c, seed)
    scale = 1.0 / math.sqrt(c["d"])
    hq = c["hkv"] * c["g"]
    if c["kind"] != "calib":
        cb, top = _codebook(c), _max_ctx(c)
        win = [[0 if _held(c, cb[k], top) == top else cb[k] for k in row] for row in _levels(c)]
    if c["kind"] == "decode":
        hist = [[x.kv(n) for n in _lengths(c)] for _ in range(_layers(c))]
        out = torch.empty((_layers(c), c["batch"], hq, c["d"]), dtype=torch.float64, device=DEV)
        for l in range(_layers(c)):
            k1, v1 = x.kv(c["batch"])
            q = x.q(c["batch"])
            for b, (k, v) in enumerate(hist[l]):
                k, v = torch.cat([k, k1[b:b + 1]]), torch.cat([v, v1[b:b + 1]])
                _attend_heads(c, out[l, b:b + 1], q[b:b + 1], k, v, k.shape[0] - 1, win[l], scale)
            hist[l] = None
        return out
    if c["kind"] == "chunk":
        k0, v0 = x.kv(c["p0"]) if c["p0"] else (None, None)
        k, v = x.kv(c["n"])
        if c["p0"]:
            k, v = torch.cat([k0, k]), torch.cat([v0, v])
        q = x.q(c["n"])
        out = torch.empty(q.shape, dtype=torch.float64, device=DEV)
        _attend_heads(c, out, q, k, v, c["p0"], win[0], scale)
        return out
    if c["kind"] == "prompt":
        out = torch.empty((_layers(c), c["n"] + 1, hq, c["d"]), dtype=torch.float64, device=DEV)
        for l in range(_layers(c)):
            k, v = x.kv(c["n"] + 1)
            _attend_heads(c, out[l], x.q(c["n"] + 1), k, v, 0, win[l], scale)
        return out
    k, v = x.kv(c["hist"])
    q = x.q(c["rows"])
    rows = torch.tensor(_rows(c), device=DEV)
    ws = [int(w) for w in c["windows"].split(",")]
    g, d = c["g"], c["d"]
    outs = torch.empty((len(ws) + 1, c["rows"], hq, d), dtype=torch.float64, device=DEV)
    for h in range(c["hkv"]):
        kh, vh = _stored(c, k[:, h]), _stored(c, v[:, h])
        qh = q[:, h * g:(h + 1) * g].reshape(-1, d).double()
        for i, w in enumerate(ws + [0]):
            o = _attend(qh, kh, vh, rows.repeat_interleave(g), w, c["sinks"], scale)
            outs[i, :, h * g:(h + 1) * g] = o.reshape(c["rows"], g, d)
    u, f = outs[:-1], outs[-1]
    scores = (u * f).sum(-1) / (u.norm(dim=-1) * f.norm(dim=-1))
    means = scores.reshape(len(ws), c["rows"], c["hkv"], g).mean(dim=(1, 3))
    return {"outs": outs, "scores": scores, "means": means}
