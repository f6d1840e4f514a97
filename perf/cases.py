"""The workloads that stand for what a serving program has this library do.

A program that serves a looped transformer (16 heads of width 128, 4 loops)
writes new tokens' latents and attends them at every loop, per layer.  The cases
are one layer's calls for decode steps, prompts and chunks appended to a longer
context, over the rank tiers of the per-head cache, the LLA-2D cache, the
rotary branch, the eviction budget, full RoPE and both data types.

``listed()`` names the cases, ``draw(rng)`` gives another of the same ranges,
``prepare`` makes a program's tensors, ``run`` is one pass through the public
entry points, ``exact`` the same in 64 bits from the definitions.
"""

import math

import torch

from paper_2607_15456_amd import lla

HEADS, WIDTH, LOOPS = 16, 128, 4
STACK = LOOPS * WIDTH
PAGE = 64

# (r_k, r_v): the long-context tiers first, then the rank sweep (rho 4.00 .. 1.33)
TIERS = ((18, 30), (36, 60), (96, 160), (120, 200), (144, 240), (192, 320), (240, 400), (288, 480))
RANKS_2D = (288, 480)


def listed():
    return [
        # The smallest call: one sequence, 512 tokens, fp32, one decode step at every loop.
        _case("decode_f32_b1_512", "decode", "f32", 1, 512, 96, 160),
        # A decode step of a batch under an eviction budget (4 + 1020 slots) at the
        # highest compression: the new token's write and its four attention calls.
        _case("step_evict_b32_1024", "step", "bf16", 32, 5003, 18, 30, sink=4, window=1020),
        # One long sequence with the decoupled rotary branch: the write of the
        # latents and the rotary key, then rotation and attention at every loop.
        _case("step_rope_b1_32k", "step", "bf16", 1, 32768, 96, 160, d_rope=64),
        # A full batch's decode at 2x compression: four calls over 2.1 GB of latents.
        _case("decode_b32_4k", "decode", "bf16", 32, 4096, 192, 320),
        # Full RoPE (keys rebuilt and rotated on read), a batch of unequal contexts.
        _case("fullrope_b8_4k", "fullrope", "bf16", 8, 4096, 192, 320, ragged=True),
        # The same at the tier that compresses least, two shorter sequences.
        _case("fullrope_b2_2k", "fullrope", "bf16", 2, 2000, 288, 480, ragged=True),
        # A prompt's write at a middle tier, with means, an odd token count.
        _case("write_b2_3001", "write", "bf16", 2, 0, 192, 320, tokens=3001, means=True),
        # A long prompt at the highest compression: the write and causal attention at every loop.
        _case("prompt_b4_8k", "prompt", "bf16", 4, 0, 18, 30, tokens=8192),
        # A short message appended to a long conversation at the 4x tier.
        _case("append_b1_300", "prompt", "bf16", 1, 7000, 96, 160, tokens=300),
        # The LLA-2D decode step of a batch: the split write and four attention calls.
        _case("step2d_b32_4k", "step2d", "bf16", 32, 4096, *RANKS_2D),
        # An LLA-2D prompt: the write over the loop x head stack and causal attention.
        _case("prompt2d_b2_4k", "prompt2d", "bf16", 2, 0, *RANKS_2D, tokens=4096),
        # An fp32 prompt of one sequence, as the parity runs use it.
        _case("prompt_f32_b1_500", "prompt", "f32", 1, 0, 96, 160, tokens=500),
    ]


def _case(name, path, dtype, batch, context, r_k, r_v, tokens=1, d_rope=0, sink=0, window=0, ragged=False,
          means=False):
    """context: tokens cached before the call's own (decode and full RoPE: tokens attended)."""
    c = {"path": path, "dtype": dtype, "batch": batch, "context": context, "tokens": tokens, "r_k": r_k, "r_v": r_v,
         "d_rope": d_rope, "sink": sink, "window": window, "ragged": ragged, "means": means}
    return {"name": name, **c} if name else c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        path = rng.choice(("decode", "decode", "step", "step", "fullrope", "write", "prompt", "prompt", "step2d",
                           "prompt2d", "f32"))
        r_k, r_v = rng.choice(TIERS)
        batch, ragged, means = _log(rng, 1, 64), rng.random() < 0.5, rng.random() < 0.3
        if path == "f32":
            if rng.random() < 0.5:
                c = _case("", "prompt", "f32", _log(rng, 1, 2), _log(rng, 1, 300) - 1, 96, 160,
                          tokens=_log(rng, 16, 600))
            else:
                c = _case("", "decode", "f32", _log(rng, 1, 4), _log(rng, 64, 4096), 96, 160, ragged=ragged)
        elif path == "decode":
            c = _case("", path, "bf16", batch, _log(rng, 100, 65536), r_k, r_v, ragged=ragged, means=means)
        elif path == "step":
            if rng.random() < 0.5:
                slots = rng.choice((260, 1024))
                c = _case("", path, "bf16", batch, _log(rng, slots + 1, 9000), r_k, r_v,
                          d_rope=rng.choice((0, 64)), sink=4, window=slots - 4)
            else:
                c = _case("", path, "bf16", batch, _log(rng, 100, 65536), r_k, r_v, d_rope=rng.choice((0, 64)))
        elif path == "fullrope":
            c = _case("", path, "bf16", _log(rng, 1, 16), _log(rng, 100, 16384), r_k, r_v, ragged=ragged, means=means)
            if c["batch"] * c["context"] > (4000 if r_k > 256 else 65536):
                continue
        elif path == "write":
            c = _case("", path, "bf16", _log(rng, 1, 4), 0, r_k, r_v, tokens=_log(rng, 65, 8192), means=means)
        elif path == "prompt":
            rope = rng.random() < 0.3
            if rope:                            # r_k + d_rope <= 95
                r_k, r_v = TIERS[0]
            c = _case("", path, "bf16", _log(rng, 1, 4), _log(rng, 1, 8192) - 1, r_k, r_v, tokens=_log(rng, 65, 8192),
                      d_rope=64 if rope else 0, means=means)
        elif path == "step2d":
            c = _case("", path, "bf16", _log(rng, 1, 48), _log(rng, 100, 8192), *RANKS_2D)
        else:
            c = _case("", path, "bf16", _log(rng, 1, 4), _log(rng, 1, 2048) - 1, *RANKS_2D, tokens=_log(rng, 65, 4096))
        if _cost(c) <= most:
            return c


def _cost(c):
    w = work(c)
    return w["bytes"] / 5e12 + w["flops"] / (4e14 if c["dtype"] == "bf16" else 4e13)


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------

def _end(c):
    """Positions used: the context and the call's own tokens (decode and full RoPE only read)."""
    return c["context"] + (0 if c["path"] in ("decode", "fullrope") else c["tokens"])


def _slots(c):
    """Slots attended by a decode call."""
    return min(_end(c), c["sink"] + c["window"]) if c["window"] else _end(c)


def _n_max(c):
    return (_slots(c) + PAGE - 1) // PAGE * PAGE


def _lens(c):
    """Attended tokens of each sequence: equal, or from the whole context down to half of it."""
    n, b = _slots(c), c["batch"]
    return [n - (n // 2) * i // b if c["ragged"] else n for i in range(b)]


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def work(c):
    """Bytes every input and output once, flops of the cheaper exact form of each contraction."""
    e, h, d = 4 if c["dtype"] == "f32" else 2, HEADS, WIDTH
    b, m, r, dr = c["batch"], c["tokens"], c["r_k"] + c["r_v"], c["d_rope"]
    kind, end = c["path"], _end(c)
    two_d = kind in ("step2d", "prompt2d")
    lat = 1 if two_d else h                     # latents per token
    byts = flops = 0
    if kind not in ("decode", "fullrope"):      # the write
        stack = h * STACK                       # stacked values of a token and axis
        byts += e * (2 * b * m * stack + (r * STACK * h) + b * m * lat * r)
        byts += e * 2 * stack if c["means"] else 0
        flops += 2 * b * m * r * (stack if two_d else h * STACK)
        byts += 2 * e * b * m * dr
    if kind in ("decode", "step", "step2d", "fullrope"):
        keys = sum(_lens(c))
        per = e * (keys * (lat * r + dr) + h * d * r) + b * h * (e * (d + dr) + 4 * d) + 2 * e * b * h * dr
        ops = 2 * h * (keys * (r + dr) + b * d * r)
        if kind == "fullrope":                  # keys rebuilt and rotated
            ops = 2 * h * (keys * (d * c["r_k"] + d + c["r_v"]) + b * d * c["r_v"])
        byts += LOOPS * per
        flops += LOOPS * ops
    elif kind in ("prompt", "prompt2d"):
        pairs = b * h * (m * c["context"] + m * (m + 1) // 2)
        absorbed = 2 * (r + dr) * pairs + 2 * b * h * m * d * r
        rebuilt = (4 * d + 2 * dr) * pairs + 2 * b * h * end * d * r
        byts += LOOPS * (e * (b * end * (lat * r + dr) + h * d * r) + b * h * m * (e * (d + dr) + 4 * d)
                         + 2 * e * b * h * m * dr)
        flops += LOOPS * min(absorbed, rebuilt)
    return {"bytes": byts, "flops": flops}


def tolerance(c):
    """About four times the error against ``exact``: fp32 sums over up to 65,536
    tokens; one bf16 rounding of written latents (a few slots of a step's cache,
    all of a prompt's) and of a rotated query; weights of 8 to 11 bits in the
    matrix products of the LLA-2D step and the prompts."""
    if c["dtype"] == "f32" or c["path"] in ("decode", "fullrope"):
        return {"rel": 1e-5}
    return {"rel": 1e-3 if c["path"] == "step" else 7e-3}


# ---------------------------------------------------------------------------
# a program's tensors
# ---------------------------------------------------------------------------

def prepare(c, seed):
    """Inputs from the seed: unit-variance stacks, latents and queries, projections
    that keep that variance; the caches hold the context and any later slots."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt = _dtype(c)

    def normal(*shape, var=1.0):
        t = torch.randn(shape, generator=gen, device="cuda", dtype=dt)
        return t if var == 1.0 else t.mul_(var ** 0.5)

    b, m, h, d, dr = c["batch"], c["tokens"], HEADS, WIDTH, c["d_rope"]
    r_k, r_v, n_max, kind = c["r_k"], c["r_v"], _n_max(c), c["path"]
    two_d = kind in ("step2d", "prompt2d")
    s = {"case": c}
    if two_d:
        s["c_k"], s["c_v"] = normal(b, n_max, r_k), normal(b, n_max // PAGE, r_v, PAGE)
    else:
        s["c_k"] = normal(b, h, n_max // PAGE, r_k, PAGE)
        s["c_v"] = normal(b, h, n_max // PAGE, r_v, PAGE)
    if kind not in ("decode", "fullrope"):
        x, w = ((b, m, h * STACK), (h * STACK,)) if two_d else ((b, m, h, STACK), (STACK,))
        lead = () if two_d else (h,)
        var = 1.0 / w[0]
        s["x_k"], s["x_v"] = normal(*x), normal(*x)
        s["w_k"], s["w_v"] = normal(*lead, r_k, *w, var=var), normal(*lead, r_v, *w, var=var)
        s["m_k"] = normal(*lead, *w) if c["means"] else None
        s["m_v"] = normal(*lead, *w) if c["means"] else None
    if kind == "write":
        return s
    rows = (m,) if kind in ("prompt", "prompt2d") else ()
    s["loops"] = []
    for _ in range(LOOPS):
        s["loops"].append({
            "q": normal(b, h, *rows, d),
            "u_k": normal(h, d, r_k, var=1.0 / r_k), "u_v": normal(h, d, r_v, var=1.0 / r_v),
            "mu_k": normal(h, d) if c["means"] else None, "mu_v": normal(h, d) if c["means"] else None,
            "q_rope": normal(b, h, *rows, dr) if dr else None,
        })
    if dr:
        s["k_rope"] = normal(b, m, 1, dr)
        s["r_cache"] = normal(b, 1, n_max // PAGE, dr, PAGE)
    if kind in ("decode", "step", "fullrope"):
        s["workspace"] = lla.new_workspace(b, h, r_v, _slots(c))
    if kind in ("step", "step2d"):              # position of the new token of every sequence
        s["pos"] = torch.full((b,), c["context"], dtype=torch.int32, device="cuda")
    if c["ragged"]:
        s["lens"] = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
    if kind == "step2d":
        s["write_ws"] = lla.new_encode_2d_workspace(b, m, h, LOOPS, d, r_k, r_v)
        s["workspace"] = torch.empty(lla.decode_2d_workspace_bytes(b, h, r_k, r_v, _end(c)), dtype=torch.uint8,
                                     device="cuda")
    if kind == "prompt":
        n = lla.prefill_workspace_bytes(dt, b, h, m, d, r_k, r_v, c["context"])
        s["workspace"] = torch.empty(n, dtype=torch.uint8, device="cuda") if n and not dr else None
    if kind == "prompt2d":
        s["workspace"] = torch.empty(lla.prefill_2d_workspace_bytes(b, h, d, _end(c)), dtype=torch.uint8,
                                     device="cuda")
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    c = s["case"]
    kind, n, evict = c["path"], _slots(c), (c["sink"], c["window"]) if c["window"] else None
    outs = []
    if kind in ("write", "step", "prompt"):
        lla.encode(s["x_k"], s["x_v"], s["w_k"], s["w_v"], s["c_k"], s["c_v"], T=LOOPS, pos0=c["context"],
                   mu_k=s["m_k"], mu_v=s["m_v"], evict=evict)
        if c["d_rope"]:
            lla.rope_write(s["k_rope"], s["r_cache"], pos0=c["context"], evict=evict)
    elif kind in ("step2d", "prompt2d"):
        lla.encode_2d(s["x_k"], s["x_v"], s["w_k"], s["w_v"], s["c_k"], s["c_v"], T=LOOPS, H=HEADS, pos0=c["context"],
                      mu_k=s["m_k"], mu_v=s["m_v"], workspace=s.get("write_ws"))
    for p in s.get("loops", ()):
        mean = {"mu_k": p["mu_k"], "mu_v": p["mu_v"]}
        args = (p["q"], s["c_k"], s["c_v"], p["u_k"], p["u_v"])
        if kind in ("decode", "step"):
            rope = {}
            if c["d_rope"]:
                rope = {"q_rope": lla.rope_rotate(p["q_rope"], pos=s["pos"]), "r_cache": s["r_cache"]}
            outs.append(lla.decode_attn(*args, n_ctx=n, ctx_len=s.get("lens"), workspace=s["workspace"], **mean, **rope))
        elif kind == "fullrope":
            outs.append(lla.decode_attn_fullrope(*args, n_ctx=n, ctx_len=s.get("lens"), workspace=s["workspace"], **mean))
        elif kind == "step2d":
            outs.append(lla.decode_attn_2d(*args, n_ctx=n, workspace=s["workspace"], **mean))
        elif kind == "prompt":
            rope = {}
            if c["d_rope"]:
                rope = {"q_rope": lla.rope_rotate(p["q_rope"], pos0=c["context"]), "r_cache": s["r_cache"]}
            outs.append(lla.prefill_attn(*args, p0=c["context"], workspace=s["workspace"], **mean, **rope))
        else:
            outs.append(lla.prefill_attn_2d(*args, p0=c["context"], workspace=s["workspace"], **mean))
    caches = [s["c_k"], s["c_v"]] + ([s["r_cache"]] if c["d_rope"] else [])
    return {"out": outs} if kind in ("decode", "fullrope") else {"out": outs, "cache": caches}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _rotate(x, pos, base=10000.0):
    """Half-split rotary embedding of x [..., f] at positions pos [...]."""
    f = x.shape[-1]
    inv = base ** (-torch.arange(f // 2, device=x.device, dtype=torch.float64) * 2.0 / f)
    a = pos.to(torch.float64)[..., None] * inv
    u, v = x[..., :f // 2], x[..., f // 2:]
    return torch.cat([u * a.cos() - v * a.sin(), v * a.cos() + u * a.sin()], -1)


def _attend(q, k, v, first=None):
    """softmax(q k^T) v; first: query m sees keys up to first + m."""
    out = torch.empty(q.shape[0], v.shape[1], dtype=torch.float64, device=q.device)
    for i in range(0, q.shape[0], 2048):
        sc = q[i:i + 2048] @ k.t()
        if first is not None:
            seen = first + i + torch.arange(sc.shape[0], device=q.device)
            sc.masked_fill_(torch.arange(k.shape[0], device=q.device) > seen[:, None], -math.inf)
        out[i:i + 2048] = torch.softmax(sc, -1) @ v
    return out


def exact(c, seed):
    s = prepare(c, seed)
    dt, kind, d, dr = _dtype(c), c["path"], WIDTH, c["d_rope"]
    b, m, n, p0 = c["batch"], c["tokens"], _slots(c), c["context"]
    two_d = kind in ("step2d", "prompt2d")
    heads = 1 if two_d else HEADS

    def slots(first, count):
        p = torch.arange(first, first + count, device="cuda")
        if not c["window"]:
            return p
        return torch.where(p < c["sink"], p, c["sink"] + (p - c["sink"]) % c["window"])

    # caches token-major [b][head] -> [n_max, r], in 64 bits; written latents unrounded
    def tokens_of(cache, paged):
        x = cache.double()
        return x.transpose(-1, -2).reshape(b, -1, _n_max(c), cache.shape[-2]) if paged else x[:, None]

    lat = {"k": tokens_of(s["c_k"], not two_d), "v": tokens_of(s["c_v"], True)}
    seen = dict(lat)
    if kind not in ("decode", "fullrope"):
        at = slots(p0, m)
        seen = {}
        for a in "kv":
            x = s["x_" + a].reshape(b, m, heads, -1)
            for h in range(heads):
                w = (s["w_" + a] if two_d else s["w_" + a][h]).double()
                mu = s["m_" + a]
                shift = 0.0 if mu is None else (mu if two_d else mu[h]).double()
                for i in range(b):
                    lat[a][i, h, at] = (x[i, :, h].double() - shift) @ w.t()
            seen[a] = lat[a].to(dt).double() if kind != "write" else None  # attention reads what the cache holds
    if dr:
        rot = s["r_cache"].double().transpose(-1, -2).reshape(b, _n_max(c), dr)
        where = torch.arange(p0, p0 + m, device="cuda")
        rot[:, slots(p0, m)] = _rotate(s["k_rope"][:, :, 0].double(), where)
        kept = rot.to(dt).double()
    outs = []
    scale = 1.0 / math.sqrt(d + dr)
    lens = _lens(c)
    for p in s.get("loops", ()):
        q = p["q"].double()
        res = torch.empty(q.shape, dtype=torch.float64, device="cuda")
        many = kind in ("prompt", "prompt2d")
        qr = None
        if dr:                                   # rotated query parts are stored in the input type
            where = p0 + torch.arange(m if many else 1, device="cuda")
            qr = p["q_rope"].double().reshape(b, HEADS, -1, dr)
            qr = _rotate(qr, where.expand(b, HEADS, -1)).to(dt).double()
        for i in range(b):
            keys = _end(c) if many else lens[i]
            for h in range(HEADS):
                ck, cv = seen["k"][i, h % heads, :keys], seen["v"][i, h % heads, :keys]
                uk, uv = p["u_k"][h].double(), p["u_v"][h].double()
                qh = q[i, h].reshape(-1, d)
                if kind == "fullrope":
                    k = ck @ uk.t()
                    if p["mu_k"] is not None:
                        k = k + p["mu_k"][h].double()
                    where = torch.arange(keys, device="cuda")
                    k = _rotate(k, where)
                    z = _attend(_rotate(qh, where[-1:]) * scale, k, cv)
                else:
                    qt = qh @ uk * scale
                    if dr:
                        qt = torch.cat([qt, qr[i, h] * scale], 1)
                        ck = torch.cat([ck, kept[i, :keys]], 1)
                    z = _attend(qt, ck, cv, p0 if many else None)
                o = z @ uv.t()
                if p["mu_v"] is not None:
                    o = o + p["mu_v"][h].double()
                res[i, h] = o.reshape(res[i, h].shape)
        outs.append(res)
    if kind in ("decode", "fullrope"):
        return {"out": outs}

    def paged(x, like):
        return x.reshape(b, -1, _n_max(c) // PAGE, PAGE, like.shape[-2]).transpose(-1, -2).reshape(like.shape)

    caches = [lat["k"][:, 0] if two_d else paged(lat["k"], s["c_k"]), paged(lat["v"], s["c_v"])]
    if dr:
        caches.append(paged(rot, s["r_cache"]))
    return {"out": outs, "cache": caches}
