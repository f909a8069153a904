"""Performance cases of the library, through its Python entry points.

Each case is one unit of work of a program that runs an LLM's short kernels
through a specialization cache: the decode chains of a stage or a whole step
(T = 1..16 tokens), the chain of a mixed-size batch or of a long prefill, and
the single ops, from the smallest call (where the launch counts) to calls that
stream hundreds of megabytes. The ranges are those of the workloads and tests
of this repository: 1-8192 tokens, rows of a few hundred to some ten thousand
elements (norm rows up to 131,072), float32 and bfloat16, contiguous tensors,
views into wider buffers (the halves of a fused gate / up projection, the heads
of a fused QKV projection, a column slice) and tensors that start one element
off a 16-byte boundary, widths that are no whole number of 16-byte vectors,
and every RoPE variant.

listed() names the cases, draw() gives others of the same ranges; prepare()
makes what the program holds before the call, run() is one pass, exact() the
same outputs in 64 bits with plain torch, work() the bytes and operations that
one pass cannot do without, tolerance() what rounding may change.
"""
import math

import torch

import paper_2609_37241_amd as tri

DEV = "cuda"
EPS = 1e-6
SCALING = dict(factor=8.0, low_freq_factor=1.0, high_freq_factor=4.0, original_max_pos=8192)
TABLE_ROWS = 8192           # rows of a caller-supplied cos / sin table
SLICE_PAD = 64              # extra columns of the buffer a row view is cut from

_ROPE_PLAIN = dict(rd=0, inter=False, pos64=False, table=False, scaling=False, qk_norm=False,
                   base=10000.0)


def _chain(name, dtype, T, H, nq, nk, hd, I, layers, entry, layout="plain", **kw):
    c = dict(name=name, op="chain", dtype=dtype, T=T, H=H, nq=nq, nk=nk, hd=hd, I=I,
             layers=layers, entry=entry, layout=layout, resident=False, outliers=False)
    c.update(_ROPE_PLAIN)
    c.update(kw)
    return c


def _rope(name, dtype, T, nq, nk, hd, layout="plain", **kw):
    c = dict(name=name, op="rope", dtype=dtype, T=T, nq=nq, nk=nk, hd=hd, layout=layout)
    c.update(_ROPE_PLAIN)
    c.update(kw)
    return c


def _rows(name, op, dtype, T, W, layout="plain", **kw):
    return dict(name=name, op=op, dtype=dtype, T=T, W=W, layout=layout, **kw)


def listed():
    return [
        # One token through a pipeline stage of 8 Llama-7B-shaped layers, the
        # argument structs built once and one call per layer from resident
        # argument blocks: the smallest calls, where only launches count.
        _chain("decode 1 token, 8 layers", "bf16", 1, 4096, 32, 32, 128, 11008, 8, "calls",
               resident=True),
        # A decode batch of 8 sequences through 32 GQA layers (Llama-3 shapes
        # and frequency scaling), captured once and replayed as a graph.
        _chain("decode 8 tokens, graph", "bf16", 8, 4096, 32, 8, 128, 14336, 32, "graph",
               scaling=True, base=500000.0),
        # A decode batch of 16 through 32 layers with per-head QK norm, in one
        # entry call; q and k are views of the fused QKV projection's output,
        # gate and up the halves of the fused gate / up projection's.
        _chain("decode 16 tokens, views", "bf16", 16, 4096, 32, 8, 128, 12288, 32, "layers",
               layout="views", qk_norm=True, base=1000000.0),
        # One call of the mixed-size stream at its largest token count, every
        # activation one element off a 16-byte boundary.
        _chain("mixed 512 tokens, offset", "bf16", 512, 4096, 32, 32, 128, 11008, 1, "calls",
               layout="offset"),
        # Prefill of 8192 tokens at hidden 8192, heavy-tailed activations: the
        # largest call, HBM bandwidth.
        _chain("prefill 8192 tokens", "bf16", 8192, 8192, 64, 8, 128, 28672, 1, "calls",
               base=500000.0, outliers=True),
        # The norm of the paper's motivating example, an ordinary Python call.
        _rows("rmsnorm f32 1024x128", "rmsnorm", "f32", 1024, 128),
        # Residual add + norm of a prompt at a ragged row length.
        _rows("residual norm 1536x4097", "residual", "bf16", 1536, 4097),
        # RoPE of a prompt of 2048 tokens with heads of 96 (six vectors a
        # half), int64 positions and the program's own cos / sin table, on
        # views of the fused QKV projection's output.
        _rope("rope heads of 96", "bf16", 2048, 32, 32, 96, layout="views", pos64=True,
              table=True),
        # SwiGLU of a prompt on the halves of the fused projection's output.
        _rows("swiglu views 4096x14336", "swiglu", "bf16", 4096, 14336, layout="views"),
        # silu at an ordinary size, an ordinary Python call.
        _rows("silu 1024x4096", "silu", "bf16", 1024, 4096),
        # Attention scores of 8 heads x 1001 queries x 1001 keys under a mask
        # that fills with -inf.
        _rows("masked fill 8008x1001", "masked_fill", "bf16", 8008, 1001),
        # Token embedding of a prompt from a 32,000-row table, int64 ids.
        _rows("embedding 8192x4096", "embedding", "bf16", 8192, 4096, n_rows=32000, ids64=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def _width(rng, lo, hi):
    """Mostly whole multiples of 64, one in four any length."""
    w = _log_int(rng, lo, hi)
    return w if rng.random() < 0.25 else max(64, w // 64 * 64)


def _rope_variant(rng):
    v = dict(_ROPE_PLAIN, base=rng.choice([1e4, 5e5, 1e6]), pos64=rng.random() < 0.3,
             qk_norm=rng.random() < 0.25, inter=rng.random() < 0.2)
    kind = rng.random()
    if kind < 0.2:
        v["scaling"] = True
    elif kind < 0.4:
        v["table"] = True
    return v


def draw(rng):
    op = rng.choice(["chain", "chain", "rmsnorm", "residual", "rope", "swiglu", "silu", "add",
                     "masked_fill", "embedding"])
    dtype = "bf16" if rng.random() < 0.75 else "f32"
    layout = rng.choice(["plain", "plain", "views", "offset"])
    es = 2 if dtype == "bf16" else 4
    most = 400 << 20            # bytes of the widest operand group, well below the prefill's
    if op in ("chain", "rope"):
        hd = rng.choice([64, 80, 96, 128, 128, 128, 256])
        nq = rng.choice([8, 16, 24, 32, 40, 64])
        nk = rng.choice([1, 2, 8, nq])
        c = dict(op=op, dtype=dtype, T=_log_int(rng, 1, 8192), nq=nq, nk=nk, hd=hd, layout=layout)
        c.update(_rope_variant(rng))
        if hd > 64 and rng.random() < 0.25:
            c["rd"] = hd // 2
        if op == "chain":
            c["H"] = _width(rng, 512, 16384)
            c["I"] = _width(rng, 688, 28672)
            c.update(layers=rng.choice([1, 2, 4]), entry=rng.choice(["calls", "layers", "graph"]),
                     resident=rng.random() < 0.3, outliers=rng.random() < 0.2)
            row = es * c["layers"] * (4 * c["H"] + (nq + 2 * nk) * hd + 3 * c["I"])
        else:
            row = es * (nq + 2 * nk) * hd
        c["T"] = max(1, min(c["T"], most // row))
        return c
    c = dict(op=op, dtype=dtype, T=_log_int(rng, 1, 8192), W=_width(rng, 128, 16384),
             layout=layout)
    if op in ("rmsnorm", "residual") and rng.random() < 0.15:
        c["W"] = _width(rng, 32768, 131072)
    if op == "embedding":
        c.update(n_rows=rng.choice([1000, 32000, 50257]), ids64=rng.random() < 0.5)
    c["T"] = max(1, min(c["T"], most // (4 * es * c["W"])))
    return c


# ---- inputs ---------------------------------------------------------------------------
_shared = None


def _cache():
    """The program's cache: one for all its calls."""
    global _shared
    if _shared is None:
        _shared = tri.SpecCache()
    return _shared


class _Draw:
    def __init__(self, case, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)
        self.dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        self.outliers = case.get("outliers", False)

    def fill(self, t):
        a = torch.randn(t.shape, generator=self.g, device=DEV)
        if self.outliers:
            a = torch.where(torch.rand(t.shape, generator=self.g, device=DEV) < 1e-3, a * 50.0, a)
        return t.copy_(a)

    def empty(self, shape, off=False):
        """A contiguous tensor, one element off a 16-byte boundary with off."""
        n = math.prod(shape)
        t = torch.zeros(n + 1 if off else n, device=DEV, dtype=self.dt)
        return t[1:].view(shape) if off else t.view(shape)

    def act(self, shape, off=False):
        return self.fill(self.empty(shape, off))

    def rows(self, T, W, layout):
        """Activation rows [T, W] in the case's layout."""
        if layout == "views":
            return self.act((T, W + SLICE_PAD))[:, :W]
        return self.act((T, W), layout == "offset")

    def weight(self, n):
        return (torch.rand((n,), generator=self.g, device=DEV) + 0.5).to(self.dt)

    def ints(self, hi, n, dt):
        return torch.randint(0, hi, (n,), generator=self.g, device=DEV, dtype=dt)


def _heads(d, case, lead):
    """q [.., T, nq, hd] and k [.., T, nk, hd] in the case's layout."""
    T, nq, nk, hd = (case[k] for k in ("T", "nq", "nk", "hd"))
    if case["layout"] == "views":                      # heads of a fused QKV output
        qkv = d.act((*lead, T, nq + 2 * nk, hd))
        return qkv[..., :nq, :], qkv[..., nq:nq + nk, :]
    off = case["layout"] == "offset"
    return d.act((*lead, T, nq, hd), off), d.act((*lead, T, nk, hd), off)


def _rope_inputs(d, case):
    T, hd = case["T"], case["hd"]
    rd = case["rd"] or hd
    s = {}
    pdt = torch.int64 if case["pos64"] else torch.int32
    s["pos"] = (d.ints(TABLE_ROWS, T, pdt) if T <= 64
                else torch.arange(T, device=DEV, dtype=pdt) + int(d.ints(1024, 1, pdt)[0]))
    if case["table"]:
        f = torch.rand((TABLE_ROWS + 1024, rd // 2), generator=d.g, device=DEV) * (2 * math.pi)
        s["table"] = torch.cat([f.cos(), f.sin()], dim=1).contiguous()
    if case["qk_norm"]:
        s["q_w"], s["k_w"] = d.weight(hd), d.weight(hd)
    plain = not (case["rd"] or case["inter"] or case["pos64"] or case["table"] or case["scaling"])
    s["ext"] = None if plain else tri.rope_ext(
        rotary_dim=case["rd"], interleaved=case["inter"], pos_int64=case["pos64"],
        scaling=SCALING if case["scaling"] else None, cos_sin=s.get("table"))
    return s


def _chain_state(d, case, cache):
    L, T, H, I = (case[k] for k in ("layers", "T", "H", "I"))
    off = case["layout"] == "offset"
    s = _rope_inputs(d, case)
    s["x"], s["residual"] = d.act((L, T, H), off), d.act((T, H), off)
    s["w"] = torch.stack([d.weight(H) for _ in range(L)])
    s["q"], s["k"] = _heads(d, case, (L,))
    if case["layout"] == "views":                      # halves of a fused gate / up output
        gu = d.act((L, T, 2 * I))
        s["gate"], s["up"] = gu[..., :I], gu[..., I:]
    else:
        s["gate"], s["up"] = d.act((L, T, I), off), d.act((L, T, I), off)
    s["y"], s["res_out"] = d.empty((L, T, H), off), d.empty((L, T, H), off)
    s["out"] = d.empty((L, T, I), off)
    s["args"] = []
    for i in range(L):
        a, _ = cache.chain_args(
            s["x"][i], s["residual"] if i == 0 else s["res_out"][i - 1], s["w"][i], s["q"][i],
            s["k"][i], s["pos"], s["gate"][i], s["up"][i], EPS, case["base"], y=s["y"][i],
            residual_out=s["res_out"][i], out=s["out"][i], q_norm_w=s.get("q_w"),
            k_norm_w=s.get("k_w"), rope=s["ext"])
        s["args"].append(a)
    if case["entry"] == "graph":
        s["graph"] = cache.build_graph(s["args"])
    return s


def prepare(case, seed):
    d, op, T = _Draw(case, seed), case["op"], case["T"]
    if op == "chain":
        # resident blocks and graphs belong to a cache of the program's part
        # that uses them
        own = case["resident"] or case["entry"] == "graph"
        cache = tri.SpecCache(resident_args=case["resident"]) if own else _cache()
        s = _chain_state(d, case, cache)
    elif op == "rope":
        cache, s = _cache(), _rope_inputs(d, case)
        s["q"], s["k"] = _heads(d, case, ())
    else:
        cache, W, layout, s = _cache(), case["W"], case["layout"], {}
        if op in ("rmsnorm", "residual"):
            s["x"], s["w"] = d.rows(T, W, layout), d.weight(W)
            if op == "residual":
                s["residual"] = d.rows(T, W, layout)
        elif op == "swiglu":
            if layout == "views":
                gu = d.act((T, 2 * W))
                s["gate"], s["up"] = gu[:, :W], gu[:, W:]
            else:
                s["gate"], s["up"] = d.rows(T, W, layout), d.rows(T, W, layout)
        elif op == "embedding":
            s["x"] = d.rows(case["n_rows"], W, layout)
            s["ids"] = d.ints(case["n_rows"], T, torch.int64 if case["ids64"] else torch.int32)
        else:
            s["x"] = d.rows(T, W, layout)
            if op == "add":
                s["b"] = d.rows(T, W, layout)
            elif op == "masked_fill":
                m = torch.rand((T, W + (SLICE_PAD if layout == "views" else 0)), generator=d.g,
                               device=DEV) < 0.3
                s["mask"] = m[:, :W]
    s["case"], s["cache"] = case, cache
    return s


def run(s):
    case, cache = s["case"], s["cache"]
    op = case["op"]
    if op == "chain":
        if case["entry"] == "graph":
            s["graph"].launch()
        elif case["entry"] == "layers":
            cache.decode_chain_layers(s["args"])
        else:
            for a in s["args"]:
                cache.decode_chain_args(a)
        return {k: s[k] for k in ("y", "res_out", "q", "k", "out")}
    if op == "rope":
        if s["ext"] is not None:
            return cache.rope(s["q"], s["k"], s["pos"], case["base"], s["ext"], q_w=s.get("q_w"),
                              k_w=s.get("k_w"), eps=EPS)
        if case["qk_norm"]:
            return cache.qk_norm_rope(s["q"], s["k"], s["pos"], s["q_w"], s["k_w"], case["base"],
                                      EPS)
        return cache.rope_qk(s["q"], s["k"], s["pos"], case["base"])
    if op == "rmsnorm":
        return cache.rmsnorm(s["x"], s["w"], EPS)
    if op == "residual":
        return cache.residual_rmsnorm(s["x"], s["residual"], s["w"], EPS)
    if op == "swiglu":
        return cache.swiglu(s["gate"], s["up"])
    if op == "silu":
        return cache.silu(s["x"])
    if op == "add":
        return cache.add(s["x"], s["b"])
    if op == "masked_fill":
        return cache.masked_fill(s["x"], s["mask"], float("-inf"))
    return cache.embedding(s["x"], s["ids"])


# ---- the same in 64 bits ----------------------------------------------------------------
def _norm64(x, w):
    x = x.double()
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + float(torch.tensor(EPS))) * w.double()


def _angles64(case, s):
    """(cos, sin) [T, rd/2]: of the float32 product of the position and the
    float32 inverse frequency, as the op defines the angle, or the table's."""
    rd = case["rd"] or case["hd"]
    if case["table"]:
        row = s["table"][s["pos"].long().clamp(0, s["table"].shape[0] - 1)].double()
        return row[:, :rd // 2], row[:, rd // 2:]
    i = torch.arange(rd // 2, device=DEV, dtype=torch.float64)
    inv = torch.pow(torch.tensor(case["base"], dtype=torch.float64, device=DEV), -2.0 * i / rd)
    inv = inv.float()
    if case["scaling"]:
        f = inv.double()
        wave, omax = 2 * math.pi / f, SCALING["original_max_pos"]
        lo, hi = SCALING["low_freq_factor"], SCALING["high_freq_factor"]
        smooth = (omax / wave - lo) / (hi - lo)
        mid = (1 - smooth) * f / SCALING["factor"] + smooth * f
        f = torch.where(wave < omax / hi, f, torch.where(wave > omax / lo, f / SCALING["factor"],
                                                         mid))
        inv = f.float()
    th = (s["pos"].float()[:, None] * inv[None, :]).double()
    return th.cos(), th.sin()


def _rotate64(v, w, case, cs):
    """Heads v [.., T, n, hd] after the optional head norm and the rotation."""
    rd = case["rd"] or case["hd"]
    v = _norm64(v, w) if w is not None else v.double()
    c, n = cs[0][:, None, :], cs[1][:, None, :]
    out = v.clone()
    if case["inter"]:
        a, b = v[..., 0:rd:2], v[..., 1:rd:2]
        out[..., 0:rd:2], out[..., 1:rd:2] = a * c - b * n, b * c + a * n
    else:
        a, b = v[..., :rd // 2], v[..., rd // 2:rd]
        out[..., :rd // 2], out[..., rd // 2:rd] = a * c - b * n, b * c + a * n
    return out


def _silu64(g):
    g = g.double()
    return g / (1 + torch.exp(-g))


def exact(case, seed):
    s = prepare(case, seed)
    op = case["op"]
    if op in ("chain", "rope"):
        cs = _angles64(case, s)
        q = _rotate64(s["q"], s.get("q_w"), case, cs)
        k = _rotate64(s["k"], s.get("k_w"), case, cs)
        if op == "rope":
            return q, k
        y, ro, r = [], [], s["residual"]
        for i in range(case["layers"]):
            ro.append(s["x"][i].double() + r.double())
            r = (s["x"][i].float() + r.float()).to(r.dtype)     # the norm is of the rounded sum
            y.append(_norm64(r, s["w"][i]))
        out = _silu64(s["gate"]).mul_(s["up"])
        return {"y": torch.stack(y), "res_out": torch.stack(ro), "q": q, "k": k, "out": out}
    if op == "rmsnorm":
        return _norm64(s["x"], s["w"])
    if op == "residual":
        h = (s["x"].float() + s["residual"].float()).to(s["x"].dtype)
        return _norm64(h, s["w"]), s["x"].double() + s["residual"].double()
    if op == "swiglu":
        return _silu64(s["gate"]).mul_(s["up"])
    if op == "silu":
        return _silu64(s["x"])
    if op == "add":
        return s["x"].double() + s["b"].double()
    if op == "masked_fill":
        return s["x"].double().masked_fill(s["mask"], float("-inf"))
    return s["x"].double()[s["ids"].long()]


# ---- bytes, operations, tolerances ---------------------------------------------------------
def work(case):
    es, T, op = (2 if case["dtype"] == "bf16" else 4), case["T"], case["op"]
    if op in ("chain", "rope"):
        L = case.get("layers", 1)
        hd, rd = case["hd"], case["rd"] or case["hd"]
        n = T * (case["nq"] + case["nk"])
        touched = hd if case["qk_norm"] else rd       # a plain rotation leaves the rest alone
        by = 2 * n * touched * es
        by += T * rd * 4 if case["table"] else 0
        by += 2 * hd * es if case["qk_norm"] else 0
        fl = n * (3 * rd + (4 * hd if case["qk_norm"] else 0))
        if op == "chain":
            H, I = case["H"], case["I"]
            by += (4 * T * H + H + 3 * T * I) * es
            fl += T * (5 * H + 6 * I)
        return {"bytes": L * by + T * (8 if case["pos64"] else 4), "flops": L * fl}
    n = T * case["W"]
    if op == "rmsnorm":
        return {"bytes": (2 * n + case["W"]) * es, "flops": 4 * n}
    if op == "residual":
        return {"bytes": (4 * n + case["W"]) * es, "flops": 5 * n}
    if op == "embedding":
        # rows drawn twice are read once
        rows = case["n_rows"] * (1 - (1 - 1 / case["n_rows"]) ** T)
        return {"bytes": (rows * case["W"] + n) * es + T * (8 if case["ids64"] else 4), "flops": 0}
    by = {"swiglu": 3 * es, "silu": 2 * es, "add": 3 * es, "masked_fill": 2 * es + 1}[op] * n
    return {"bytes": by, "flops": {"swiglu": 6, "silu": 5, "add": 1, "masked_fill": 0}[op] * n}


def tolerance(case):
    # Sums of one rounding, selections and copies have one right answer. The
    # others are computed in float32 and rounded once: in bfloat16 an output
    # is 1.7e-3 (2-norm) off its 64-bit value, at most one step (2^-7 of the
    # value) where a correct implementation rounds the other way; in float32
    # the paths measure up to 7e-8 (2-norm) and 1.3e-6 (largest) off theirs.
    if case["op"] in ("add", "masked_fill", "embedding"):
        return "exact"
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 3e-7, "max": 6e-6}
