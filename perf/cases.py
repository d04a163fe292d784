"""The calls whose speed matters to a user of the selective-recompute prefill.

A request is served layer by layer: its chunks' caches are staged to the GPU,
one check layer selects the tokens to recompute, and every later layer runs
the decoder steps on the selected tokens around a reuse-mode blend.  The cases
below take the public entry points through that work, from a request of about
a thousand tokens to the 124k-token contexts, in the head layouts of the
models the method is evaluated on: 32 query / 8 kv heads with hidden size 4096
and a feed-forward width of 14336, 28 / 4 heads with 3584 and 18944, one GPU's
share of an 8-way split by kv head (4 / 1 heads), and a small 8 / 2 layout.

Kinds of case:

* ``check``: ``kvc_blend_prefill_layer`` on the check layer (adjust,
  deviation, selection, blend, attention); ratio 1 recomputes every row;
* ``reuse``: the same call on a later layer, on the compact selected rows;
* ``front``: the check layer's projections: norm of every row, keys of every
  row, then norm (gathering), Q/K/V and RoPE of the selected rows;
* ``decoder``: a whole reuse layer, norm to down projection;
* ``mlp``: the feed-forward half of a layer;
* ``select``: ``kvc_select_tokens``, the check layer's selection alone;
* ``stage``: ``kvc_stage_layers``, one layer's chunk caches from pinned host
  memory, merged and adjusted.
"""
import math
import random

import torch

import paper_2609_09768_amd as K

D = 128
THETA = 500000.0
EPS = 1e-5
NOISE = 0.1
DEV = "cuda:0"
BF = torch.bfloat16

# query heads, kv heads, hidden size, feed-forward width
MODELS = {
    "small": (8, 2, 1024, 3584),
    "llama8b": (32, 8, 4096, 14336),
    "qwen7b": (28, 4, 3584, 18944),
    "llama8b-tp8": (4, 1, 4096, 1792),
}


def listed():
    return [
        # the shortest request: five dependent steps of a few microseconds
        {"name": "check-1k-small", "kind": "check", "model": "small", "reused": 1024, "chunks": 4, "docs": 0,
         "query": 64, "ratio": 0.15},
        # a short retrieval context
        {"name": "check-4k", "kind": "check", "model": "llama8b", "reused": 4000, "chunks": 16, "docs": 0,
         "query": 96, "ratio": 0.15},
        # retrieval documents of mixed length with zero-K/V separators
        {"name": "check-32k-docs", "kind": "check", "model": "llama8b", "reused": 32000, "chunks": 0, "docs": 175,
         "query": 256, "ratio": 0.15},
        # the long-context request the method is meant for
        {"name": "check-124k", "kind": "check", "model": "llama8b", "reused": 124000, "chunks": 16, "docs": 0,
         "query": 256, "ratio": 0.15},
        # a layer recomputed in full (the layers before the check layer), seven query heads to a kv head
        {"name": "full-6k-qwen", "kind": "check", "model": "qwen7b", "reused": 5997, "chunks": 7, "docs": 0,
         "query": 131, "ratio": 1.0},
        # later layers at a low recompute ratio
        {"name": "reuse-32k-5pc", "kind": "reuse", "model": "llama8b", "reused": 32000, "chunks": 16, "docs": 0,
         "query": 256, "ratio": 0.05},
        # one GPU's share of a later layer of the 124k request
        {"name": "reuse-124k-tp8", "kind": "reuse", "model": "llama8b-tp8", "reused": 124000, "chunks": 16, "docs": 0,
         "query": 256, "ratio": 0.15},
        # the check layer's projections
        {"name": "front-16k", "kind": "front", "model": "llama8b", "reused": 16000, "chunks": 16, "docs": 0,
         "query": 200, "ratio": 0.15},
        # whole later layers, short and long
        {"name": "decoder-4k", "kind": "decoder", "model": "llama8b", "reused": 4000, "chunks": 16, "docs": 0,
         "query": 96, "ratio": 0.15},
        {"name": "decoder-32k", "kind": "decoder", "model": "llama8b", "reused": 32000, "chunks": 16, "docs": 0,
         "query": 256, "ratio": 0.15},
        # the feed-forward half on the selection of a short request, an odd row count
        {"name": "mlp-217-qwen", "kind": "mlp", "model": "qwen7b", "rows": 217},
        # one layer of a document context from pinned host memory
        {"name": "stage-32k-docs", "kind": "stage", "model": "llama8b", "reused": 32000, "chunks": 0, "docs": 175,
         "query": 256, "ratio": 0.15},
    ]


def draw(rng):
    """One more case: any kind and model, 512 to 48k reused tokens (96k for one GPU's share)."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["check", "check", "reuse", "front", "decoder", "decoder", "mlp", "select", "stage"])
    model = rng.choice(["small", "llama8b", "llama8b", "qwen7b", "llama8b-tp8"])
    if kind == "mlp":
        return {"kind": kind, "model": model, "rows": log_int(100, 12000)}
    reused = log_int(512, 96000 if model == "llama8b-tp8" else 48000)
    full = kind == "check" and rng.random() < 0.2
    if full:
        reused = min(reused, 5000 + log_int(1, 4000))
    docs = rng.choice([0, 0, rng.randint(40, 400)])
    chunks = 0 if docs else rng.randint(1, min(32, reused // 64))
    ratio = 1.0 if full else round(rng.choice([0.05, 0.15, 0.15, 0.3, rng.uniform(0.02, 0.4)]), 3)
    return {"kind": kind, "model": model, "reused": reused, "chunks": chunks, "docs": docs,
            "query": rng.randint(1, 300), "ratio": ratio}


# ---- shapes ------------------------------------------------------------------
def _chunks(case):
    """Chunk lengths and zero-K/V flags: nearly even chunks, or documents
    between two-token separators (lognormal lengths of the given mean)."""
    total = case["reused"]
    if not case["docs"]:
        n = case["chunks"]
        return [total // n + (i < total % n) for i in range(n)], None
    rng = random.Random(total * 1000 + case["docs"])
    mu = math.log(case["docs"]) - 0.18
    lens, zero, left = [], [], total - 2
    while left > 0:
        n = int(min(512, max(16, round(rng.lognormvariate(mu, 0.6)))))
        if left - n - 2 < 20:
            n = left - 2
        lens += [2, n]
        zero += [1, 0]
        left -= n + 2
    return lens + [2], zero + [1]


def _counts(case):
    n_r, n_q = case["reused"], case["query"]
    return n_r, n_r + n_q, math.floor(case["ratio"] * n_r) + n_q


def _layout(case):
    hq, hkv = MODELS[case["model"]][:2]
    lens, zero = _chunks(case)
    return K.Layout(lens, case["query"], hq, hkv, D, THETA, None, None, zero)


# ---- inputs --------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV)


def _inv_freq():
    return THETA ** (-torch.arange(0, D, 2, dtype=torch.float64, device=DEV) / D)


def _rope(x, pos):
    """Half-split RoPE of x [rows, heads, D] at positions pos, in x's type."""
    ang = pos.to(torch.float64)[:, None] * _inv_freq()
    c, s = torch.cos(ang).to(x.dtype)[:, None, :], torch.sin(ang).to(x.dtype)[:, None, :]
    a, b = x[..., :D // 2], x[..., D // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _positions(lens, n_rows):
    """Chunk-local position of every row (query rows keep their global one)."""
    pos = torch.arange(n_rows, device=DEV)
    start = torch.tensor([0] + lens, device=DEV).cumsum(0)[:-1]
    n_r = sum(lens)
    pos[:n_r] -= torch.repeat_interleave(start, torch.tensor(lens, device=DEV))
    return pos


def _zero_rows(lens, zero):
    rows, r = [], 0
    for n, z in zip(lens, zero or [0] * len(lens)):
        if z:
            rows += range(r, r + n)
        r += n
    return torch.tensor(rows, dtype=torch.int64, device=DEV)


def _caches(case, g):
    """Cached keys at chunk-local positions, recomputed keys, cached and
    recomputed values: per-channel scales from lognormal(0, 0.5), recomputed
    = cached + 10 % noise, zeros in the separators' cached rows."""
    hkv = MODELS[case["model"]][1]
    n_r, n_rows, _ = _counts(case)
    lens, zero = _chunks(case)
    z = _zero_rows(lens, zero)
    raw = _randn(g, n_rows, hkv, D) * torch.exp(0.5 * _randn(g, hkv, D))
    k_src = _rope(raw, _positions(lens, n_rows)).to(BF)
    k_fresh = _rope(raw + NOISE * _randn(g, n_rows, hkv, D), torch.arange(n_rows, device=DEV)).to(BF)
    raw = _randn(g, n_rows, hkv, D) * torch.exp(0.5 * _randn(g, hkv, D))
    v_cache = raw.to(BF)
    v_fresh = (raw + NOISE * _randn(g, n_rows, hkv, D)).to(BF)
    k_src[z] = 0
    v_cache[z] = 0
    return {"k_src": k_src[:n_r].clone(), "k_fresh": k_fresh, "v_cache": v_cache, "v_fresh": v_fresh}


def _queries(case, g, rows):
    hq = MODELS[case["model"]][0]
    return _rope(_randn(g, len(rows), hq, D) * torch.exp(0.5 * _randn(g, hq, D)), rows).to(BF)


def _selection(case, g):
    """An earlier check layer's selection: rows spread over the context, then the query rows."""
    n_r, n_rows, n_sel = _counts(case)
    k = n_sel - case["query"]
    top = torch.rand(n_r, generator=g, device=DEV).topk(k).indices.sort().values
    return torch.cat([top, torch.arange(n_r, n_rows, device=DEV)]).to(torch.int32)


def _weights(case, g):
    hq, hkv, hid, inter = MODELS[case["model"]]
    w = lambda n, k: (_randn(g, n, k) / math.sqrt(k)).to(BF)  # noqa: E731
    gamma = lambda: (1 + 0.1 * _randn(g, hid)).to(BF)  # noqa: E731
    kind = case["kind"]
    out = {}
    if kind in ("front", "decoder"):
        out.update(g1=gamma(), wqkv=w((hq + 2 * hkv) * D, hid))
    if kind == "decoder":
        out.update(wo=w(hid, hq * D))
    if kind in ("decoder", "mlp"):
        out.update(g2=gamma(), wgu=w(2 * inter, hid), wd=w(hid, inter))
    return out


def _inputs(case, seed):
    g, kind = _gen(seed), case["kind"]
    hid = MODELS[case["model"]][2]
    s = {}
    if kind == "mlp":
        s["x"] = _randn(g, case["rows"], hid).to(BF)
        s.update(_weights(case, g))
        return s
    n_r, n_rows, n_sel = _counts(case)
    if kind != "front":
        s.update(_caches(case, g))
    if kind == "check":
        s["q"] = _queries(case, g, torch.arange(n_rows, device=DEV))
    elif kind in ("reuse", "decoder", "front"):
        s["sel"] = _selection(case, g)
    if kind in ("reuse", "decoder"):
        sel = s["sel"].long()
        s["k_fresh"], s["v_fresh"] = s["k_fresh"][sel], s["v_fresh"][sel]
    if kind == "reuse":
        s["q"] = _queries(case, g, sel)
    elif kind == "front":
        s["x"] = _randn(g, n_rows, hid).to(BF)
        s.update(_weights(case, g))
    elif kind == "decoder":
        s["x"] = _randn(g, n_sel, hid).to(BF)
        s.update(_weights(case, g))
        del s["k_fresh"], s["v_fresh"]
    elif kind == "stage":
        del s["k_fresh"], s["v_fresh"]
    return s


def _empty(*shape, dtype=BF):
    return torch.empty(shape, dtype=dtype, device=DEV)


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    hq, hkv, hid, inter = MODELS[case["model"]]
    s["case"] = case
    if kind == "mlp":
        n = case["rows"]
        s.update(h=_empty(n, hid), gu=_empty(n, 2 * inter), a=_empty(n, inter), out=_empty(n, hid))
        return s
    n_r, n_rows, n_sel = _counts(case)
    if kind != "front":
        L = s["L"] = _layout(case)
        nb = K.kvc_plan_bytes(L)
        s["plan"] = K.kvc_plan_upload(L, _empty(nb, dtype=torch.uint8), nb)
        s["wb"] = K.kvc_blend_workspace(L) + K.kvc_attention_workspace(n_sel, hq, hkv, D)
        s["ws"] = _empty(s["wb"], dtype=torch.uint8)
    if kind in ("check", "select"):
        s["sel"] = _empty(n_sel, dtype=torch.int32)
    if kind in ("check", "reuse", "decoder"):
        s.update(k_cache=torch.zeros(n_rows, hkv, D, dtype=BF, device=DEV), attn=_empty(n_sel, hq, D),
                 lse=_empty(n_sel, hq, dtype=torch.float32))
    if kind == "select":
        s["k_cache"] = _empty(n_r, hkv, D)
    if kind == "front":
        s.update(h_all=_empty(n_rows, hid), y_all=_empty(n_rows, hkv * D), k_all=_empty(n_rows, hkv, D),
                 h=_empty(n_sel, hid), res=_empty(n_sel, hid), y=_empty(n_sel, (hq + 2 * hkv) * D),
                 q=_empty(n_sel, hq, D), k=_empty(n_sel, hkv, D), v=_empty(n_sel, hkv, D))
        s["wk"] = s["wqkv"][hq * D:(hq + hkv) * D]
    elif kind == "decoder":
        s.update(h=_empty(n_sel, hid), y=_empty(n_sel, (hq + 2 * hkv) * D), q=_empty(n_sel, hq, D),
                 k=_empty(n_sel, hkv, D), v=_empty(n_sel, hkv, D), x1=_empty(n_sel, hid),
                 gu=_empty(n_sel, 2 * inter), a=_empty(n_sel, inter), out=_empty(n_sel, hid))
    elif kind == "stage":
        # each document's cache where the document store put it: one pinned
        # arena, documents in shuffled order; separators have no cache
        lens, zero = _chunks(case)
        order = [i for i in range(len(lens)) if not (zero and zero[i])]
        random.Random(seed).shuffle(order)
        start = [0]
        for n in lens:
            start.append(start[-1] + n)
        s["k_host"], s["v_host"] = [], []
        for src, name in ((s.pop("k_src"), "k_host"), (s.pop("v_cache")[:n_r], "v_host")):
            arena = torch.empty((sum(lens[i] for i in order), hkv, D), dtype=BF, pin_memory=True)
            arena.copy_(torch.cat([src[start[i]:start[i + 1]] for i in order]))
            at, ptr = 0, [None] * len(lens)
            for i in order:
                ptr[i] = arena[at:at + lens[i]]
                at += lens[i]
            s[name] = ptr
        s.update(k_cache=_empty(n_r, hkv, D), v_cache=_empty(n_r, hkv, D))
    return s


# ---- one pass --------------------------------------------------------------------
def _mlp(s, x, n, hid, inter):
    K.kvc_rms_norm(x, n, None, n, hid, s["g2"], EPS, s["h"])
    K.kvc_projection(n, 2 * inter, hid, s["h"], n, None, s["wgu"], None, s["gu"])
    K.kvc_swiglu(s["gu"], n, inter, s["a"])
    K.kvc_projection(n, hid, inter, s["a"], n, None, s["wd"], x, s["out"])


def run(s):
    case = s["case"]
    kind = case["kind"]
    hq, hkv, hid, inter = MODELS[case["model"]]
    if kind == "mlp":
        _mlp(s, s["x"], case["rows"], hid, inter)
        return s["out"]
    n_r, n_rows, n_sel = _counts(case)
    if kind in ("check", "reuse"):
        K.kvc_blend_prefill_layer(s["L"], s["plan"], kind == "check", case["ratio"], s["k_src"], s["k_cache"],
                                  s["v_cache"], s["q"], s["k_fresh"], s["v_fresh"], s["sel"], n_sel, s["attn"],
                                  s["lse"], s["ws"], s["wb"])
        return {k: s[k] for k in ("k_cache", "v_cache", "sel", "attn", "lse")}
    if kind == "select":
        K.kvc_select_tokens(s["L"], s["plan"], case["ratio"], s["k_src"], s["k_cache"], s["k_fresh"], s["sel"],
                            n_sel, s["ws"], s["wb"])
        return {"k_cache": s["k_cache"], "sel": s["sel"]}
    if kind == "stage":
        K.kvc_stage_layers(s["L"], s["plan"], 1, s["k_host"], s["v_host"], [s["k_cache"]], [s["v_cache"]])
        return {"k_cache": s["k_cache"], "v_cache": s["v_cache"]}
    if kind == "front":
        K.kvc_rms_norm(s["x"], n_rows, None, n_rows, hid, s["g1"], EPS, s["h_all"])
        K.kvc_projection(n_rows, hkv * D, hid, s["h_all"], n_rows, None, s["wk"], None, s["y_all"])
        K.kvc_qkv_rope(s["y_all"], n_rows, 0, hkv, 0, D, None, THETA, None, s["k_all"], None)
        K.kvc_rms_norm(s["x"], n_rows, s["sel"], n_sel, hid, s["g1"], EPS, s["h"], s["res"])
        K.kvc_projection(n_sel, (hq + 2 * hkv) * D, hid, s["h"], n_sel, None, s["wqkv"], None, s["y"])
        K.kvc_qkv_rope(s["y"], n_sel, hq, hkv, hkv, D, s["sel"], THETA, s["q"], s["k"], s["v"])
        return {k: s[k] for k in ("k_all", "res", "q", "k", "v")}
    K.kvc_rms_norm(s["x"], n_sel, None, n_sel, hid, s["g1"], EPS, s["h"])
    K.kvc_projection(n_sel, (hq + 2 * hkv) * D, hid, s["h"], n_sel, None, s["wqkv"], None, s["y"])
    K.kvc_qkv_rope(s["y"], n_sel, hq, hkv, hkv, D, s["sel"], THETA, s["q"], s["k"], s["v"])
    K.kvc_blend_prefill_layer(s["L"], s["plan"], False, case["ratio"], s["k_src"], s["k_cache"], s["v_cache"],
                              s["q"], s["k"], s["v"], s["sel"], n_sel, s["attn"], None, s["ws"], s["wb"])
    K.kvc_projection(n_sel, hid, hq * D, s["attn"], n_sel, None, s["wo"], s["x"], s["x1"])
    _mlp(s, s["x1"], n_sel, hid, inter)
    return {k: s[k] for k in ("k_cache", "v_cache", "attn", "out")}


# ---- what a pass cannot do without ---------------------------------------------
def _mlp_work(n, hid, inter):
    return {"bytes": 2 * (2 * n * hid + 3 * hid * inter), "flops": 6.0 * n * hid * inter}


def work(case):
    hq, hkv, hid, inter = MODELS[case["model"]]
    kind = case["kind"]
    if kind == "mlp":
        return _mlp_work(case["rows"], hid, inter)
    n_r, n_rows, n_sel = _counts(case)
    row = 2 * hkv * D  # bytes of one K or V row
    if kind == "select":
        return {"bytes": 3 * n_r * row + 4 * n_sel, "flops": 0}
    if kind == "stage":
        return {"bytes": 2 * 2 * n_r * row, "flops": 0}
    if kind == "front":
        nqkv = (hq + 2 * hkv) * D
        return {"bytes": 2 * (n_rows * hid + nqkv * hid + n_sel * (hid + nqkv)) + n_rows * row,
                "flops": 2.0 * hid * (n_rows * hkv * D + n_sel * nqkv)}
    # causal by position: the selected rows spread over the reused ones, then the query rows
    visible = (n_sel - case["query"]) * (n_r + 1) / 2 + case["query"] * (n_r + n_rows + 1) / 2
    flops = 4.0 * hq * D * visible
    # the shift's read and write, K and V for the attention, the blended rows, Q and out
    move = 2 * n_r * row + n_rows * row + 4 * n_sel * row + 4 * n_sel * hq * D
    if kind == "check":
        extra = n_r * row if case["ratio"] < 1 else 0
        return {"bytes": move + extra + 4 * n_sel * (1 + hq), "flops": flops}
    if kind == "reuse":
        return {"bytes": move + 4 * n_sel * (1 + hq), "flops": flops}
    m = _mlp_work(n_sel, hid, inter)
    nqkv = (hq + 2 * hkv) * D
    # queries, attention output and recomputed rows need not leave the chip between steps
    return {"bytes": m["bytes"] + 2 * n_r * row + n_rows * row + 2 * n_sel * row + 2 * hid * (nqkv + hq * D),
            "flops": m["flops"] + flops + 2.0 * n_sel * hid * (nqkv + hq * D)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("select", "stage"):
        return "exact"  # keys rounded once, values copied, rows by exact comparison
    if kind in ("check", "reuse"):
        # bf16 outputs (2^-9 each) of bf16-rounded weights; the rest is exact
        return {"rel": 0.01, "max": 0.06, "differ": 0.0}
    # four to nine bf16 roundings in a row
    return {"rel": 0.015, "max": 0.1, "differ": 0.0}


# ---- the same in float64 -----------------------------------------------------------
def _to_bf16(x):
    """float64 to bfloat16 values (nearest, ties to even, one rounding), as float64."""
    f = x.float()
    tie = (f.view(torch.int32) & 0xFFFF) == 0x8000
    away = torch.copysign(torch.full_like(f, math.inf), f)
    towards = torch.where(f.double().abs() < x.abs(), away, torch.zeros_like(f))
    return torch.where(tie & (f.double() != x), torch.nextafter(f, towards), f).to(BF).double()


def _shifted(case, k_src):
    lens, zero = _chunks(case)
    n_r = case["reused"]
    delta = torch.arange(n_r, device=DEV) - _positions(lens, n_r)
    out = torch.empty(k_src.shape, dtype=torch.float64, device=DEV)
    for a in range(0, n_r, 16384):
        out[a:a + 16384] = _to_bf16(_rope(k_src[a:a + 16384].double(), delta[a:a + 16384]))
    return out


def _attention(q, k, v, pos):
    """Causal GQA by position in float64: (out, lse), one kv head and block of queries at a time."""
    n, hq, _ = q.shape
    hkv = k.shape[1]
    grp = hq // hkv
    out = torch.empty(n, hq, D, dtype=torch.float64, device=DEV)
    lse = torch.empty(n, hq, dtype=torch.float64, device=DEV)
    step = max(1, int(2.5e8 // (k.shape[0] * grp)))
    for g in range(hkv):
        kt, vg = k[:, g].double().t().contiguous(), v[:, g].double().contiguous()
        for a in range(0, n, step):
            b = min(n, a + step)
            m = int(pos[a:b].max()) + 1
            s = q[a:b, g * grp:(g + 1) * grp].double().reshape(-1, D) @ kt[:, :m]
            s *= 1 / math.sqrt(D)
            hide = torch.arange(m, device=DEV)[None, :] > pos[a:b].repeat_interleave(grp)[:, None]
            s.masked_fill_(hide, -math.inf)
            l = torch.logsumexp(s, dim=1)
            s -= l[:, None]
            o = s.exp_() @ vg[:m]
            out[a:b, g * grp:(g + 1) * grp] = o.reshape(b - a, grp, D)
            lse[a:b, g * grp:(g + 1) * grp] = l.reshape(b - a, grp)
    return out, lse


def _norm(x, gamma):
    x = x.double()
    return x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + EPS) * gamma.double()


def _mlp_exact(s, x, inter):
    gu = _norm(x, s["g2"]) @ s["wgu"].double().t()
    gate, up = gu[:, :inter], gu[:, inter:]
    return x + (gate * torch.sigmoid(gate) * up) @ s["wd"].double().t()


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    hq, hkv, hid, inter = MODELS[case["model"]]
    if kind == "mlp":
        return _mlp_exact(s, s["x"].double(), inter)
    n_r, n_rows, n_sel = _counts(case)
    if kind == "front":
        sel = s["sel"].long()
        h = _norm(s["x"], s["g1"])
        wk = s["wqkv"][hq * D:(hq + hkv) * D].double()
        y = (h[sel] @ s["wqkv"].double().t()).reshape(n_sel, hq + 2 * hkv, D)
        return {"k_all": _rope((h @ wk.t()).reshape(n_rows, hkv, D), torch.arange(n_rows, device=DEV)),
                "res": s["x"][sel].double(), "q": _rope(y[:, :hq], sel), "k": _rope(y[:, hq:hq + hkv], sel),
                "v": y[:, hq + hkv:]}
    kc = torch.zeros(n_rows, hkv, D, dtype=torch.float64, device=DEV)
    kc[:n_r] = _shifted(case, s["k_src"])
    if kind == "stage":
        return {"k_cache": kc[:n_r], "v_cache": s["v_cache"][:n_r].double()}
    if kind in ("check", "select"):
        if case["ratio"] >= 1:
            sel = torch.arange(n_rows, device=DEV)
        else:
            d = torch.cat([((f.double() - c) ** 2).sum((1, 2))
                           for f, c in zip(s["k_fresh"][:n_r].split(16384), kc[:n_r].split(16384))])
            top = torch.sort(d, descending=True, stable=True).indices[:n_sel - case["query"]].sort().values
            sel = torch.cat([top, torch.arange(n_r, n_rows, device=DEV)])
        if kind == "select":
            return {"k_cache": kc[:n_r], "sel": sel.to(torch.int32)}
        fresh, q = (s["k_fresh"][sel].double(), s["v_fresh"][sel].double()), s["q"][sel]
    else:
        sel = s["sel"].long()
        if kind == "reuse":
            fresh, q = (s["k_fresh"].double(), s["v_fresh"].double()), s["q"]
        else:
            y = (_norm(s["x"], s["g1"]) @ s["wqkv"].double().t()).reshape(n_sel, hq + 2 * hkv, D)
            q = _rope(y[:, :hq], sel)
            fresh = (_rope(y[:, hq:hq + hkv], sel), y[:, hq + hkv:])
    vc = s["v_cache"].double()
    kc[sel], vc[sel] = fresh
    out, lse = _attention(q, kc, vc, sel)
    if kind != "decoder":
        return {"k_cache": kc, "v_cache": vc, "sel": sel.to(torch.int32), "attn": out, "lse": lse}
    x1 = s["x"].double() + out.reshape(n_sel, hq * D) @ s["wo"].double().t()
    return {"k_cache": kc, "v_cache": vc, "attn": out, "out": _mlp_exact(s, x1, inter)}
