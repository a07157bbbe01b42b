"""The work that users of this library have it do, as cases that can be timed and compared.

Every case goes through the public entry points of ``paper_2607_15621_amd.fsx`` and is described by plain values:

* ``tick``     one control tick of the action expert (``expert_forward``): all layers and the head over the standing cache
* ``clip``     the same forward over the blocks of one training clip, which share one agent's cache (CACHE_SHARED)
* ``loop``     the deployment loop: one append of the slow system's rows on its own stream, then four ticks
* ``append``   the slow system's rows into the cache rings, as a copy or encoded into an fp8 cache
* ``backbone`` the slow system itself: the backbone's incremental forward over new tokens (``Backbone.append``)

The full-size expert has 32 layers, width 512, 32 heads of 128 and a SwiGLU of 2,048; the backbone has LLaMA-7B's shapes
(32 layers, width 4,096, SwiGLU 11,008).  Weights are seeded normals of variance 1 / fan-in, cached rows and tokens
N(0, 1), fp8 caches hold E4M3 codes with one scale amax / 448 per (agent, layer, head).
"""

import math

import numpy as np
import torch

from paper_2607_15621_amd import fsx

EXPERT = dict(n_layers=32, d=512, H=32, Dh=128, F=2048)
EXPERT_F32 = dict(n_layers=2, d=64, H=4, Dh=32, F=256)
BACKBONE = dict(n_layers=32, d=4096, H=32, Dh=128, F=11008)
T, N_OUT, HIDDEN, EPS, ROPE = 10, 10, 512, 1e-6, 10000.0
TEXT, PER_FRAME = 64, 4  # cached rows of the instruction and of one frame
BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64


def _tick(name, dtype="bf16", cache="bf16", batch=1, rows=224, ragged=False, frame=0, token_major=False, query_head=False,
          hidden=True, spare=0):
    return dict(name=name, kind="tick", dtype=dtype, cache=cache, batch=batch, rows=rows, ragged=ragged, frame=frame,
                token_major=token_major, query_head=query_head, hidden=hidden, spare=spare)


def listed():
    return [
        # the smallest expert, in fp32: bring-up and numerics work, where launches are all there is
        _tick("tick_small_fp32", dtype="fp32", cache="fp32", rows=40),
        # the deployed tick: one vehicle, 64 instruction rows and 40 frames in the cache, waypoints only
        _tick("tick_40_frames", hidden=False),
        # a few vehicles on one device with the paper's head, an fp8 cache in the backbone's own layout, uneven histories
        _tick("tick_4_agents_fp8", cache="fp8", batch=4, rows=1491, ragged=True, token_major=True, query_head=True, spare=21),
        # a long history, and the current frame's tokens take part as queries
        _tick("tick_64_frame_tokens", rows=4096, frame=64),
        # sixteen vehicles (or simulator instances) served together
        _tick("tick_16_agents", batch=16, rows=1024, spare=16),
        # the longest histories, which fit as fp8
        _tick("tick_8_agents_fp8_long", cache="fp8", batch=8, rows=16001, ragged=True, spare=383),
        # the training form: 40 frames' blocks of one clip over its shared cache, each two frames stale
        dict(name="clip_40_blocks", kind="clip", blocks=40, stale=2),
        # deployment: every fourth tick the slow system's four rows come in (full rings, the oldest rows go)
        dict(name="loop_4_ticks_fp8", kind="loop", cache="fp8", batch=2, rows=224, new=4),
        # the append of sixteen vehicles by itself
        dict(name="append_16_agents", kind="append", cache="bf16", source="bf16", batch=16, rows=224, new=4,
             token_major=False),
        # the slow system: one frame's tokens of one vehicle, ...
        dict(name="backbone_1_agent", kind="backbone", cache="bf16", batch=1, new=4, rows=224, hidden=False),
        # ... of sixteen, ...
        dict(name="backbone_16_agents", kind="backbone", cache="bf16", batch=16, new=4, rows=1024, hidden=True),
        # ... and the start of eight episodes: the instruction's tokens into empty rings
        dict(name="backbone_prefill_8x64", kind="backbone", cache="bf16", batch=8, new=TEXT, rows=0, hidden=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tick"] * 7 + ["small", "clip", "loop", "append"] + ["backbone"] * 3)
    if kind == "small":
        c = _tick("", dtype="fp32", cache="fp32", batch=rng.randint(1, 4), rows=rng.randint(0, 256), ragged=rng.random() < 0.5,
                  spare=rng.randint(0, 9))
    elif kind == "tick":
        cache = rng.choice(["bf16", "bf16", "fp8"])
        batch = _log(rng, 1, 16)
        frame = rng.choice([0, 0, 0, rng.randint(1, 64)])
        frame = min(frame, 400 // batch - T)
        rows = min(_log(rng, 24, 16384), (64000 if cache == "fp8" else 32000) // batch)
        c = _tick("", cache=cache, batch=batch, rows=rows, ragged=rng.random() < 0.5, frame=frame,
                  token_major=rng.random() < 0.4, query_head=rng.random() < 0.3, hidden=rng.random() < 0.7,
                  spare=rng.randint(0, 64))
    elif kind == "clip":
        c = dict(kind="clip", blocks=rng.randint(8, 40), stale=rng.randint(1, 4))
    elif kind == "loop":
        c = dict(kind="loop", cache=rng.choice(["fp8", "bf16"]), batch=rng.randint(1, 4), rows=rng.randint(160, 1100),
                 new=rng.randint(1, 8))
    elif kind == "append":
        cache = rng.choice(["bf16", "fp8"])
        c = dict(kind="append", cache=cache, source=cache if cache == "bf16" else rng.choice(["bf16", "fp32"]),
                 batch=_log(rng, 1, 16), rows=rng.randint(160, 300), new=rng.randint(1, 12), token_major=rng.random() < 0.5)
    else:
        batch, new = _log(rng, 1, 16), _log(rng, 1, TEXT)
        new = min(new, 512 // batch)
        cache, rows = rng.choice(["bf16", "bf16", "fp8"]), _log(rng, 64, 1024)
        rows = max(8 * new, rows) if cache == "fp8" else rng.choice([0, max(new, rows)])
        c = dict(kind="backbone", cache=cache, batch=batch, new=new, rows=rows, hidden=rng.random() < 0.5)
    c.pop("name", None)
    return c


# ------------------------------------------------------------------------------------------------ shapes and inputs

def _shape(c):
    return BACKBONE if c["kind"] == "backbone" else (EXPERT_F32 if c.get("dtype") == "fp32" else EXPERT)


def _lengths(c):
    """Cached rows of each agent."""
    if c["kind"] == "clip":
        return [TEXT + PER_FRAME * max(0, j - c["stale"]) for j in range(1, c["blocks"] + 1)]
    rows, n = c["rows"], c["batch"]
    if not c.get("ragged"):
        return [rows] * n
    return [rows - rows * ((29 * b) % 64) // 64 for b in range(n)]


def _capacity(c):
    """Ring slots: what the agents hold and some; appends run on full rings, a prefill into an empty one of 40 frames."""
    if c["kind"] == "clip":
        return TEXT + PER_FRAME * c["blocks"]
    if c["kind"] == "backbone" and c["rows"] == 0:
        return TEXT + PER_FRAME * 40
    return max(c["rows"] + c.get("spare", 0), c.get("new", 0), 1)


def _starts(c, cap):
    """Ring start of each agent; appends and loops run on rings that have wrapped before."""
    return [(37 * b + 11) % cap if c["kind"] in ("append", "loop", "backbone") and c["rows"] else 0 for b in range(len(_lengths(c)))]


def _gen(seed, *key):
    g = torch.Generator(device="cuda")
    x = int(seed)
    for k in key:
        x = (x * 1000003 + int(k) + 12345) & 0x3FFFFFFFFFFFFF
    g.manual_seed(x)
    return g


def _normal(g, shape, std=1.0, dtype=BF16):
    x = torch.randn(shape, generator=g, device="cuda", dtype=F32)
    return (x * std if std != 1.0 else x).to(dtype)


def _dtype(name):
    return {"bf16": BF16, "fp32": F32, "fp8": torch.uint8}[name]


def _layer(c, seed, l):
    """Layer l's weights: variance 1 / fan-in, norm gains about 1."""
    s, dt, g = _shape(c), _dtype(c.get("dtype", "bf16")), _gen(seed, 1, l)
    d, A, F = s["d"], s["H"] * s["Dh"], s["F"]
    w = lambda n, k: _normal(g, (n, k), 1.0 / math.sqrt(k), dt)  # noqa: E731
    out = {"wq": w(A, d), "wk": w(A, d), "wv": w(A, d), "wo": w(d, A), "w_gate": w(F, d), "w_up": w(F, d), "w_down": w(d, F)}
    for n in ("attn_norm", "ffn_norm"):
        out[n] = 1.0 + 0.1 * torch.randn(d, generator=g, device="cuda")
    return out


def _head(c, seed):
    s, dt, g = _shape(c), _dtype(c.get("dtype", "bf16")), _gen(seed, 2)
    d = s["d"]
    final = 1.0 + 0.1 * torch.randn(d, generator=g, device="cuda")
    if c.get("query_head"):
        return final, {"w1": _normal(g, (HIDDEN, d), d ** -0.5, dt), "b1": _normal(g, (HIDDEN,), 0.02, F32),
                       "w2": _normal(g, (2, HIDDEN), HIDDEN ** -0.5, dt), "b2": _normal(g, (2,), 0.02, F32)}
    return final, _normal(g, (N_OUT, d), d ** -0.5, dt)


def _tokens(c, seed, k=0):
    s, dt = _shape(c), _dtype(c.get("dtype", "bf16"))
    n = len(_lengths(c))
    rows = c["new"] if c["kind"] == "backbone" else T + c.get("frame", 0)
    return _normal(_gen(seed, 3, k), (n, rows, s["d"]), 1.0, dt)


def _rope_base(c):
    return 0.0 if c.get("query_head") else ROPE  # the paper's own expert has learned positions, part of its tokens


def _slab(c, seed, b, l, kv, n):
    """Rows 0 .. n-1 of (agent b, layer l), [H][n][Dh], and the fp8 scales [H] (None otherwise)."""
    s, cache = _shape(c), c.get("cache", "bf16")
    x = _normal(_gen(seed, 4, b, l, kv), (s["H"], n, s["Dh"]), 1.0, F32 if cache == "fp32" else BF16)
    if cache != "fp8":
        return x, None
    x = x.float()
    scale = x.abs().amax(dim=(1, 2)).clamp(min=1e-6) / 448.0
    return (x / scale[:, None, None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8), scale


def _cache(c, seed):
    """The rings, and their descriptor; a state's own copy of the ring's start, length and position."""
    s, lens, cap, cache = _shape(c), _lengths(c), _capacity(c), c.get("cache", "bf16")
    shared, major = c["kind"] == "clip", bool(c.get("token_major"))
    held = [max(lens)] if shared else lens
    starts = _starts(c, cap)
    nb, nl, H, Dh = len(held), s["n_layers"], s["H"], s["Dh"]
    shape = (nb, nl, cap, H, Dh) if major else (nb, nl, H, cap, Dh)
    k, v = (torch.zeros(shape, dtype=_dtype(cache), device="cuda") for _ in range(2))
    ks, vs = ((torch.ones((nb, nl, H), device="cuda") for _ in range(2)) if cache == "fp8" else (None, None))
    for b, n in enumerate(held):
        slots = (torch.arange(n, device="cuda") + starts[b]) % cap
        for l in range(nl):
            for kv, (t, sc) in enumerate(((k, ks), (v, vs))):
                if n or cache == "fp8":
                    x, scale = _slab(c, seed, b, l, kv, max(n, 64))
                    if scale is not None:
                        sc[b, l] = scale
                    x = x[:, :n]
                    if major:
                        t[b, l].index_copy_(0, slots, x.transpose(0, 1).contiguous())
                    elif starts[b] == 0:
                        t[b, l, :, :n] = x
                    else:
                        t[b, l].index_copy_(1, slots, x)
    layout = (fsx.CACHE_TOKEN_MAJOR if major else 0) | (fsx.CACHE_SHARED if shared else 0)
    kind = {"bf16": fsx.BF16, "fp32": fsx.F32, "fp8": fsx.FP8_E4M3}[cache]
    desc = fsx.CacheDesc(k, v, kind, nl, H, Dh, cap, lens, positions=lens, starts=starts, k_scale=ks, v_scale=vs, layout=layout)
    return dict(desc=desc, k=k, v=v, k_scale=ks, v_scale=vs)


def _new_rows(c, seed):
    """The slow system's rows in the cache's layout: keys and values."""
    s, n, B = _shape(c), c["new"], c["batch"]
    shape = (B, s["n_layers"], n, s["H"], s["Dh"]) if c.get("token_major") else (B, s["n_layers"], s["H"], n, s["Dh"])
    dt = _dtype(c.get("source", "bf16"))
    return [_normal(_gen(seed, 5, kv), shape, 1.0, dt) for kv in (0, 1)]


def _expert(c, seed):
    s, f32 = _shape(c), c.get("dtype") == "fp32"
    final, head = _head(c, seed)
    cfg = fsx.make_cfg(s["n_layers"], s["d"], s["H"], s["Dh"], s["F"], T, N_OUT, len(_lengths(c)), c.get("frame", 0),
                       fsx.F32 if f32 else fsx.BF16, _rope_base(c), EPS,
                       head_kind=fsx.HEAD_QUERY_MLP if c.get("query_head") else fsx.HEAD_MEAN_LINEAR,
                       head_hidden=HIDDEN if c.get("query_head") else 0)
    return fsx.expert_create(cfg, [_layer(c, seed, l) for l in range(s["n_layers"])], final, head)


def prepare(case, seed):
    c = dict(case)
    s, n = _shape(c), len(_lengths(c))
    st = dict(case=c, **_cache(c, seed))
    if c["kind"] == "append":
        st["rows"] = _new_rows(c, seed)
    elif c["kind"] == "backbone":
        cfg = fsx.BackboneCfg(s["n_layers"], s["d"], s["H"], s["Dh"], s["F"], c["new"], n, fsx.BF16, ROPE, EPS)
        st["backbone"] = fsx.Backbone(cfg, [_layer(c, seed, l) for l in range(s["n_layers"])])
        st["tokens"] = _tokens(c, seed)
        st["hidden"] = torch.zeros((s["n_layers"], n, c["new"], s["d"]), device="cuda") if c["hidden"] else None
    else:
        st["expert"] = _expert(c, seed)
        if c["kind"] == "loop":
            st["rows"] = _new_rows(c, seed)
            st["tokens"] = [_tokens(c, seed, k) for k in range(4)]
            st["waypoints"] = [torch.zeros((n, N_OUT), device="cuda") for _ in range(4)]
            st["stream"] = torch.cuda.Stream()
            st["loop"] = fsx.Loop(st["expert"], st["desc"], 4, torch.cuda.current_stream(), st["stream"])
        else:
            st["tokens"] = _tokens(c, seed)
            st["waypoints"] = torch.zeros((n, N_OUT), device="cuda")
            want = c.get("hidden", True)
            st["hidden"] = torch.zeros((s["n_layers"], n, T + c.get("frame", 0), s["d"]), device="cuda") if want else None
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return st


def run(state):
    c = state["case"]
    if c["kind"] == "append":
        k, v = state["rows"]
        if c["cache"] == "fp8":
            fsx.cache_append_rows_quantize(state["desc"], k, v, fsx.F32 if c["source"] == "fp32" else fsx.BF16, c["new"])
        else:
            fsx.cache_append_rows(state["desc"], k, v, c["new"])
        return {"k": state["k"], "v": state["v"]}
    if c["kind"] == "backbone":
        desc = state["desc"]
        if not c["rows"]:  # the start of an episode: the rings are empty
            desc.start[:] = 0
            desc.len[:] = 0
            desc.pos[:] = 0
        state["backbone"].append(desc, state["tokens"], c["batch"], c["new"], state["hidden"])
        out = {"k": state["k"], "v": state["v"]}
        return dict(out, hidden=state["hidden"]) if c["hidden"] else out
    if c["kind"] == "loop":
        k, v = state["rows"]
        state["loop"].append(k, v, fsx.BF16, c["new"])
        for tok, wp in zip(state["tokens"], state["waypoints"]):
            state["loop"].tick(tok, c["batch"], 0, wp)
        return {"waypoints": state["waypoints"], "k": state["k"], "v": state["v"]}
    n = state["waypoints"].shape[0]
    fsx.expert_forward(state["expert"], state["desc"], state["tokens"], n, c.get("frame", 0), state["waypoints"], state["hidden"])
    out = {"waypoints": state["waypoints"]}
    return out if state["hidden"] is None else dict(out, hidden=state["hidden"])


# ------------------------------------------------------------------------------------------------ what a pass needs

def work(case):
    c = dict(case)
    s, lens = _shape(c), _lengths(c)
    nl, d, A, F, n = s["n_layers"], s["d"], s["H"] * s["Dh"], s["F"], len(lens)
    es = {"bf16": 2, "fp32": 4, "fp8": 1}[c.get("cache", "bf16")]
    ws = 4 if c.get("dtype") == "fp32" else 2
    row = nl * 2 * A * es  # one cached token
    new = 0
    if c["kind"] in ("append", "loop"):
        new = n * c["new"] * nl * 2 * A * ({"fp32": 4}.get(c.get("source"), 2) + es)
        if c["kind"] == "append":
            return {"bytes": new, "flops": 0}
    S = c["new"] if c["kind"] == "backbone" else T + c.get("frame", 0)
    M, per = n * S, nl * (4 * A * d + 3 * F * d)
    held = max(lens) if c["kind"] == "clip" else sum(lens)  # shared rows are read once
    seen = sum(S * (L + (S + 1) / 2 if c["kind"] == "backbone" else L + S) for L in lens)
    head = 0 if c["kind"] == "backbone" else (HIDDEN * d + 2 * HIDDEN if c.get("query_head") else N_OUT * d)
    nbytes = (per + head) * ws + held * row + M * d * ws
    if c["kind"] == "backbone":
        nbytes += M * row
    if c.get("hidden", c["kind"] == "clip"):
        nbytes += nl * M * d * 4
    flops = 2 * M * per + 4 * nl * A * seen
    times = 4 if c["kind"] == "loop" else 1
    return {"bytes": times * nbytes + new, "flops": times * flops}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"
    if case.get("dtype") == "fp32":
        return {"rel": 1e-5}
    # 32 layers with bf16 operands between them: 0.009 off the 64-bit result, here as in the per-phase launches (the ten
    # waypoints of one agent up to 0.017); codes of an fp8 cache may fall on the other side of a rounding
    return {"rel": 0.03, "max": 0.2, "differ": 0.01 if case["kind"] == "backbone" else 0.0}


# ------------------------------------------------------------------------------------------------ the same in 64 bits

def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g.to(F64)


def _rot(x, pos, base):
    """x [n][H][Dh] rotated by the positions pos [n]: pairs (j, j + Dh/2)."""
    if base <= 0:
        return x
    half = x.shape[-1] // 2
    ang = pos[:, None] * torch.pow(torch.tensor(base, dtype=F64, device=x.device),
                                   -torch.arange(half, dtype=F64, device=x.device) / half)[None]
    cs, sn = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cs - b * sn, b * cs + a * sn], -1)


def _attend(q, k, v, causal_from=None):
    """q [n][H][Dh] over k, v [H][R][Dh]; causal_from: query i sees rows up to causal_from + i."""
    qh = q.permute(1, 2, 0).contiguous()
    sc = torch.matmul(k, qh) / math.sqrt(q.shape[-1])  # [H][R][n]
    if causal_from is not None:
        r = torch.arange(k.shape[1], device=q.device)[:, None]
        sc = sc.masked_fill(r > causal_from + torch.arange(q.shape[0], device=q.device)[None], -math.inf)
    p = torch.softmax(sc, 1).transpose(1, 2).contiguous()
    return torch.matmul(p, v).transpose(0, 1).reshape(q.shape[0], -1)


def _rows_of(c, cache, b, l, kv, length):
    """Agent b's valid rows of layer l in order, [H][length][Dh], in 64 bits."""
    t, sc = (cache["v"], cache["v_scale"]) if kv else (cache["k"], cache["k_scale"])
    b = 0 if c["kind"] == "clip" else b
    cap = _capacity(c)
    slots = (torch.arange(length, device="cuda") + int(cache["desc"].start[b])) % cap
    x = t[b, l].index_select(0, slots).transpose(0, 1) if c.get("token_major") else t[b, l].index_select(1, slots)
    if sc is not None:
        return x.contiguous().view(torch.float8_e4m3fn).to(F64) * sc[b, l].to(F64)[:, None, None]
    return x.to(F64)


def _forward(c, seed, cache, tokens, lens, pos, wants_hidden, keep=None):
    """The layers over tokens [n][S][d]; keep(l, b, k, v): the new rows, [S][H][Dh].  Returns the last and every layer's output."""
    s, base = _shape(c), ROPE if c["kind"] == "backbone" else _rope_base(c)
    H, Dh, d = s["H"], s["Dh"], s["d"]
    n, S = tokens.shape[:2]
    causal = c["kind"] == "backbone"
    h, hidden = tokens.to(F64).reshape(n * S, d), []
    where = torch.cat([p + torch.arange(S, dtype=F64, device="cuda") for p in pos])
    for l in range(s["n_layers"]):
        w = {k: x.to(F64) for k, x in _layer(c, seed, l).items()}
        x = _rms(h, w["attn_norm"])
        q, k = (_rot((x @ w[m].T).reshape(-1, H, Dh), where, base) for m in ("wq", "wk"))
        v = (x @ w["wv"].T).reshape(-1, H, Dh)
        a = []
        for b in range(n):
            i = slice(b * S, (b + 1) * S)
            rows = [torch.cat([_rows_of(c, cache, b, l, kv, lens[b]), y[i].transpose(0, 1)], 1) for kv, y in ((0, k), (1, v))]
            a.append(_attend(q[i], rows[0], rows[1], lens[b] if causal else None))
            if keep:
                keep(l, b, k[i], v[i])
        h = h + torch.cat(a) @ w["wo"].T
        x = _rms(h, w["ffn_norm"])
        h = h + (torch.nn.functional.silu(x @ w["w_gate"].T) * (x @ w["w_up"].T)) @ w["w_down"].T
        if wants_hidden:
            hidden.append(h.reshape(n, S, d))
    return h.reshape(n, S, d), torch.stack(hidden) if wants_hidden else None


def _waypoints(c, seed, h):
    final, head = _head(c, seed)
    if not c.get("query_head"):
        return _rms(h[:, :T], final).mean(1) @ head.to(F64).T
    x = _rms(h[:, T - N_OUT // 2:T], final)
    u = torch.nn.functional.gelu(x @ head["w1"].to(F64).T + head["b1"].to(F64))
    return (u @ head["w2"].to(F64).T + head["b2"].to(F64)).reshape(h.shape[0], N_OUT)


def _put_rows(c, cache, k, v):
    """The new rows [B][n_layers][H][new][Dh] into the rings (the bytes that the cache then holds)."""
    desc, cap = cache["desc"], _capacity(c)
    for b in range(c["batch"]):
        slots = (torch.arange(c["new"], device="cuda") + int(desc.start[b] + desc.len[b])) % cap
        for t, sc, x in ((cache["k"], cache["k_scale"], k), (cache["v"], cache["v_scale"], v)):
            y = x[b]
            if sc is not None:
                y = (y.float() / sc[b][:, :, None, None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
            t[b].index_copy_(2, slots, y)
        full = int(desc.len[b]) + c["new"] - cap
        desc.start[b] = (int(desc.start[b]) + max(0, full)) % cap
        desc.len[b] = min(cap, int(desc.len[b]) + c["new"])
        desc.pos[b] += c["new"]


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "append":
        return None  # copies and codes: nothing is rounded but by definition
    cache, lens = _cache(c, seed), _lengths(c)
    desc = cache["desc"]
    if c["kind"] == "loop":
        _put_rows(c, cache, *_new_rows(c, seed))
        lens = [int(x) for x in desc.len]
        got = [_waypoints(c, seed, _forward(c, seed, cache, _tokens(c, seed, k), lens, [float(p) for p in desc.pos], False)[0])
               for k in range(4)]
        return {"waypoints": got, "k": None, "v": None}
    pos = [float(p) for p in desc.pos]
    if c["kind"] != "backbone":
        h, hidden = _forward(c, seed, cache, _tokens(c, seed), lens, pos, c.get("hidden", True))
        out = {"waypoints": _waypoints(c, seed, h)}
        return out if hidden is None else dict(out, hidden=hidden)
    new = {}

    def keep(l, b, k, v):
        new[l, b] = (k.transpose(0, 1), v.transpose(0, 1))

    hidden = _forward(c, seed, cache, _tokens(c, seed), lens, pos, c["hidden"], keep)[1]
    out = {"k": None, "v": None}
    if c["cache"] == "bf16":
        cap = _capacity(c)
        slots = [(torch.arange(c["new"], device="cuda") + int(desc.start[b] + desc.len[b])) % cap for b in range(c["batch"])]
        for kv, name in enumerate(("k", "v")):
            out[name] = cache.pop(name).to(F64)
            for (l, b), rows in new.items():
                out[name][b, l].index_copy_(1, slots[b], rows[kv])
    return out if hidden is None else dict(out, hidden=hidden)
