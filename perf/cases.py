"""Performance cases of the library: what a serving program asks of one routed attention layer (or a few of them).

A case is a dict of plain values; `prepare` makes the device tensors such a program holds before the call, `run` is one
pass through the C ABI binding, `exact` the same outputs in float64 with torch alone.

Kinds of case
  router   one flux_router call: pooled boundary tokens -> logits and mode bytes.
  decode   one decode step of a stack of layers: flux_attn_decode_append per layer.
  ring     the same step of sparse layers on ring caches: flux_kv_append_ring + flux_attn_decode_ring per layer.
  prefill  new tokens of a batch behind what is cached already (0 = a whole prompt): flux_kv_append +
           flux_attn_prefill per layer.
  xa       prefill of whole prompts in the XA sparse mode: flux_kv_append, flux_xa_select and
           flux_attn_prefill_blocksparse.

A pass that appends first takes the lengths back by the number of appended tokens (what speculative decoding does with a
rejected token), so it can be repeated on the same state.

Lists are texts: "lens" = comma-separated lengths, "modes" = one word per layer, words separated by "/", one letter per
sequence (F = full attention, S = sparse) or one letter for all.
"""
import functools
import math

import torch

from paper_2604_07394_amd import binding as F

DEV = "cuda"
MAX_PREFILL_FLOPS = 8.8e12      # the listed 32768-token FA prefill: no drawn case asks for more
MAX_DECODE_BYTES = 4.4e9        # the listed 8 x 131072 FA decode
XA_HOT = 0.08                   # share of key blocks the structured XA input makes every query look at


def _ints(text):
    return [int(x) for x in text.split(",")]


def _text(values):
    return ",".join(str(v) for v in values)


def listed():
    sa8b = {"n_sink": 128, "window": 4096, "sa_block": 0}
    return [
        # the Layer Router of an 8B model (hidden 4096, inner 256, 100 + 100 boundary tokens) on a ragged batch
        {"name": "router_b4", "kind": "router", "hidden": 4096, "inner": 256, "pool": 100, "lens": "1000,4099,8192,16384"},
        # smallest call: single-user chat, one token against a short context, four layers of an 8B model, half routed SA
        {"name": "decode_b1_2k", "kind": "decode", "hq": 32, "hkv": 8, "d": 128, "lens": "2001", "modes": "F/S/F/S", "fp32": 0, **sa8b},
        # continuous batching: 32 requests of very different lengths in flight, modes routed per sequence, 28/4 heads
        {"name": "decode_b32_ragged", "kind": "decode", "hq": 28, "hkv": 4, "d": 128, "n_sink": 64, "window": 2048, "sa_block": 0, "fp32": 0,
         "lens": _text(513 + (i * 2657) % 7919 for i in range(32)), "modes": "FSFFSFSS" * 4 + "/" + "SFFSFSSF" * 4},
        # long-context decode, batch 8 x 131072 cached tokens: a layer routed SA ...
        {"name": "decode_b8_sa_128k", "kind": "decode", "hq": 32, "hkv": 8, "d": 128, "lens": _text([131071] * 8), "modes": "S/S", "fp32": 0, **sa8b},
        # ... and a layer routed FA: the largest decode call
        {"name": "decode_b8_fa_128k", "kind": "decode", "hq": 32, "hkv": 8, "d": 128, "lens": _text([131071] * 8), "modes": "F", "fp32": 0, **sa8b},
        # sparse layers that keep only their ring of rows (sparse-decode residency), 16 requests
        {"name": "ring_b16", "kind": "ring", "hq": 28, "hkv": 4, "d": 128, "n_sink": 64, "window": 2048, "sa_block": 0, "fp32": 0,
         "lens": _text(1500 + 4097 * i for i in range(16)), "modes": "S/S/S/S"},
        # smallest prefill: a 512-token prompt, 8/2 heads of 64, four layers FA SA FA SA, fp32 output
        {"name": "prefill_tiny_d64", "kind": "prefill", "hq": 8, "hkv": 2, "d": 64, "n_sink": 16, "window": 128, "sa_block": 0, "fp32": 1,
         "new": "512", "past": "0", "modes": "F/S/F/S"},
        # ordinary serving prefill: a ragged batch of short prompts, modes routed per sequence
        {"name": "prefill_ragged_2k", "kind": "prefill", "hq": 32, "hkv": 8, "d": 128, "fp32": 0, **sa8b,
         "new": "129,777,2048,3001,511", "past": "0,0,0,0,0", "modes": "FSFFS"},
        # a further turn of four conversations: some hundred new tokens each behind a long cached context
        {"name": "prefill_turns_16k", "kind": "prefill", "hq": 32, "hkv": 8, "d": 128, "fp32": 0, **sa8b,
         "new": "200,333,150,512", "past": "16200,9001,24000,12345", "modes": "FFSF"},
        # a long prompt (32768 tokens), block-granular SA layer with per-head input scales
        {"name": "prefill_sa_32k", "kind": "prefill", "hq": 32, "hkv": 8, "d": 128, "fp32": 0, "n_sink": 128, "window": 4096, "sa_block": 64,
         "new": "32768", "past": "0", "modes": "S"},
        # the same prompt in a layer routed FA: the largest prefill call
        {"name": "prefill_fa_32k", "kind": "prefill", "hq": 32, "hkv": 8, "d": 128, "fp32": 0, **sa8b,
         "new": "32768", "past": "0", "modes": "F"},
        # the XA sparse mode on a prompt whose attention has structure (a few hot key blocks per KV head)
        {"name": "xa_16k", "kind": "xa", "hq": 32, "hkv": 8, "d": 128, "fp32": 0, "lens": "16384", "threshold": 0.9},
    ]


# ---- sizes ----------------------------------------------------------------------------------------------------------

def _modes(case, batch):
    """Per layer, per sequence: True = FA."""
    return [[(w * batch if len(w) == 1 else w)[b] == "F" for b in range(batch)] for w in case["modes"].split("/")]


def _geom(case):
    b = max(1, case["sa_block"])
    return b, -(-case["n_sink"] // b) * b, -(-case["window"] // b)


def _window_lo(case, i):
    """First key of the window of the query at position i (block-granular when sa_block says so)."""
    b, _, wb = _geom(case)
    return max(0, (i // b - wb + 1) * b)


def _visible(case, i, fa):
    """Keys that the query at position i attends to."""
    if fa:
        return i + 1
    sink = min(_geom(case)[1], i + 1)
    return sink + max(0, i + 1 - max(sink, _window_lo(case, i)))


def _visible_sum(case, lo, hi, fa):
    """Sum of _visible over the positions lo .. hi - 1."""
    if fa:
        return (hi * (hi + 1) - lo * (lo + 1)) // 2
    return sum(_visible(case, i, False) for i in range(lo, hi))


def _rows_read(case, lo, hi, fa):
    """Cached rows that the queries at positions lo .. hi - 1 attend to between them."""
    if fa or hi <= lo:
        return hi
    sink = min(_geom(case)[1], hi)
    return sink + max(0, hi - max(sink, _window_lo(case, lo)))


def work(case):
    kind = case["kind"]
    if kind == "router":
        lens = _ints(case["lens"])
        h, inner = case["hidden"], case["inner"]
        rows = sum(n if case["pool"] == 0 else min(n, 2 * case["pool"]) for n in lens)
        return {"bytes": 2 * rows * h + 2 * inner * (h + 2) + 9 * len(lens), "flops": rows * h + 2 * len(lens) * inner * (h + 2)}
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    o = 4 if case["fp32"] else 2
    if kind in ("decode", "ring"):
        lens = _ints(case["lens"])
        byts = flops = 0
        for layer in _modes(case, len(lens)):
            for n, fa in zip(lens, layer):
                vis = _visible(case, n, fa)                  # the appended token sits at position n
                byts += 2 * vis * hkv * d * 2 + 2 * hkv * d * 2 + hq * d * (2 + o)
                flops += 4 * vis * hq * d
        return {"bytes": byts, "flops": flops}
    if kind == "prefill":
        new, past = _ints(case["new"]), _ints(case["past"])
        byts = flops = 0
        for layer in _modes(case, len(new)):
            for n, p, fa in zip(new, past, layer):
                byts += n * hq * d * (2 + o) + 2 * 2 * n * hkv * d * 2      # q, out; new rows read and stored
                byts += 2 * max(0, _rows_read(case, p, p + n, fa) - n) * hkv * d * 2
                flops += 4 * d * hq * _visible_sum(case, p, p + n, fa)
        return {"bytes": byts, "flops": flops}
    byts = flops = 0                                         # xa
    for n in _ints(case["lens"]):
        nb = -(-n // 64)
        byts += n * hq * d * (2 + o) + 2 * 2 * n * hkv * d * 2 + hq * nb * nb
        flops += hq * (n // 16) * (n // 16 + 1) // 2 * 2 * 16 * d           # antidiagonal sums of the causal squares
        flops += 4 * d * hq * (nb * 64 * 65 // 2 + int(XA_HOT * nb * (nb - 1) / 2 * 64 * 64))   # own blocks + hot columns
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # Router: fp32 sums over bf16 inputs (2e-7 off float64).  Attention: fp32 accumulation, weights rounded to bf16 for the
    # second product (1.0e-3 .. 1.3e-3 off float64), output rounded to bf16 unless fp32 is asked for (2.1e-3).  XA: a block
    # near the threshold's cut may fall on either side of it (a few of the two million flags of a 16384-token prompt).
    if case["kind"] == "router":
        return {"rel": 2e-6, "max": 2e-5}
    rel = 5e-3 if case["fp32"] else 8e-3
    if case["kind"] == "xa":
        lens = _ints(case["lens"])
        return {"rel": rel, "max": 0.3, "differ": max(2e-5, 2 / (case["hq"] * len(lens) * (-(-max(lens) // 64)) ** 2))}
    return {"rel": rel, "max": 0.05}


# ---- inputs ---------------------------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _context():
    return F.flux_create(0)                                  # a program keeps one context


def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + salt)
    return g


def _normal(shape, g, scale=None, dim=0):
    """bf16 N(0, 1), times a scale per index of `dim`."""
    t = torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    if scale is not None:
        t.mul_(scale.to(torch.bfloat16).view([-1 if i == dim else 1 for i in range(len(shape))]))
    return t


def _scales(n, g):
    return torch.rand(n, device=DEV, generator=g) * 1.5 + 0.5


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device=DEV)


def _cu(lens):
    c = [0]
    for n in lens:
        c.append(c[-1] + n)
    return _i32(c)


def _router_inputs(case, seed):
    g = _gen(seed)
    h, inner = case["hidden"], case["inner"]
    return {"x": _normal((sum(_ints(case["lens"])), h), g), "w1": _normal((inner, h), g) * 0.02, "w2": _normal((2, inner), g) * 0.02}


def _layer_inputs(case, seed, layer, new, rows):
    """Queries, new K/V rows and a cache filled with `rows` positions, of one layer."""
    g = _gen(seed, 17 * (layer + 1))
    hq, hkv, d, t = case["hq"], case["hkv"], case["d"], sum(new)
    sq, sk, sv = _scales(hq, g), _scales(hkv, g), _scales(hkv, g)
    return {"q": _normal((t, hq, d), g, sq, 1), "k_new": _normal((t, hkv, d), g, sk, 1), "v_new": _normal((t, hkv, d), g, sv, 1),
            "k": _normal((len(new), hkv, rows, d), g, sk, 1), "v": _normal((len(new), hkv, rows, d), g, sv, 1)}


def _xa_inputs(case, seed):
    """Every query leans towards a direction of its head; the keys of a few blocks (whole columns per KV head) do too."""
    g = _gen(seed)
    hq, hkv, d, lens = case["hq"], case["hkv"], case["d"], _ints(case["lens"])
    t = sum(lens)
    u = torch.sign(torch.randn(hkv, d, device=DEV, generator=g)) * (0.8 * math.sqrt(128 / d))
    hot = torch.cat([(torch.rand(-(-n // 64), hkv, device=DEV, generator=g) < XA_HOT).repeat_interleave(64, 0)[:n] for n in lens])
    q = torch.randn(t, hq, d, device=DEV, generator=g) + u.repeat_interleave(hq // hkv, 0)
    k = torch.randn(t, hkv, d, device=DEV, generator=g) + hot[:, :, None] * u
    return {"q": q.to(torch.bfloat16), "k_new": k.to(torch.bfloat16), "v_new": _normal((t, hkv, d), g)}


def _out(case, rows):
    return torch.zeros(rows, case["hq"], case["d"], dtype=torch.float32 if case["fp32"] else torch.bfloat16, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "ctx": _context()}
    if kind == "router":
        lens = _ints(case["lens"])
        st.update(_router_inputs(case, seed), cu=_cu(lens), mode=torch.zeros(len(lens), dtype=torch.uint8, device=DEV),
                  logits=torch.zeros(len(lens), 2, dtype=torch.float32, device=DEV))
        return st
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    if kind == "xa":
        lens = _ints(case["lens"])
        nb = -(-max(lens) // 64)
        st.update(_xa_inputs(case, seed), cfg=F.attn_cfg(hq, hkv, d, 0, 1, 0.0, case["fp32"]), cu=_cu(lens), added=_i32(lens), lens=lens, nb=nb,
                  cache=F.KVCache(torch.zeros(len(lens), hkv, max(lens), d, dtype=torch.bfloat16, device=DEV),
                                  torch.zeros(len(lens), hkv, max(lens), d, dtype=torch.bfloat16, device=DEV), _i32(lens)),
                  mode=torch.zeros(len(lens), dtype=torch.uint8, device=DEV),
                  keep=torch.zeros(len(lens), hq, nb, nb, dtype=torch.uint8, device=DEV), out=_out(case, sum(lens)))
        return st
    if kind == "prefill":
        new, past = _ints(case["new"]), _ints(case["past"])
    else:
        past = _ints(case["lens"])
        new = [1] * len(past)
    total = [n + p for n, p in zip(new, past)]
    modes = _modes(case, len(new))
    _, sink, wb = _geom(case)
    window = wb * max(1, case["sa_block"])
    rows = sink + window if kind == "ring" else max(total) + 64
    kv_len = _i32([total] * len(modes))                      # what the previous pass left behind: run() takes it back first
    layers = []
    for i, fa in enumerate(modes):
        x = _layer_inputs(case, seed, i, new, rows)
        # keys any sequence of this layer attends to: all of them, or the sparse list where every sequence is SA
        bound = max(total) if any(fa) else min(max(total), sink + window)
        layers.append({"q": x["q"], "k_new": x["k_new"], "v_new": x["v_new"], "cache": F.KVCache(x["k"], x["v"], kv_len[i]), "bound": bound,
                       "mode": torch.tensor(fa, dtype=torch.uint8, device=DEV), "out": _out(case, sum(new))})
    st.update(cfg=F.attn_cfg(hq, hkv, d, case["n_sink"], case["window"], 0.0, case["fp32"], case["sa_block"]), layers=layers, kv_len=kv_len,
              added=_i32(new), cu=_cu(new), t=sum(new), max_new=max(new), max_total=max(total), sink=sink, window=window)
    return st


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "router":
        F.flux_router(ctx, st["x"], st["cu"], st["mode"].shape[0], case["hidden"], case["pool"], st["w1"], None, st["w2"], None, case["inner"],
                      st["mode"], st["logits"])
        return {"logits": st["logits"], "mode": st["mode"]}
    hkv, d, cfg = case["hkv"], case["d"], st["cfg"]
    if kind == "xa":
        c, n = st["cache"], max(st["lens"])
        c.kv_len.sub_(st["added"])
        F.flux_kv_append(ctx, c, hkv, d, st["k_new"], st["v_new"], st["cu"], sum(st["lens"]), n)
        F.flux_xa_select(ctx, cfg, st["q"], st["cu"], n, n, c, 16, case["threshold"], st["keep"], st["nb"], st["nb"])
        F.flux_attn_prefill_blocksparse(ctx, cfg, st["q"], st["cu"], n, n, c, st["mode"], st["keep"], case["hq"], st["nb"], st["nb"], st["out"])
        return {"out": st["out"], "keep": st["keep"], "k": c.k, "v": c.v, "len": c.kv_len}
    st["kv_len"].sub_(st["added"])
    for x in st["layers"]:
        if kind == "decode":
            F.flux_attn_decode_append(ctx, cfg, x["q"], x["k_new"], x["v_new"], x["bound"], x["cache"], x["mode"], x["out"])
        elif kind == "ring":
            F.flux_kv_append_ring(ctx, x["cache"], hkv, d, st["sink"], st["window"], x["k_new"], x["v_new"], st["cu"], st["t"], 1)
            F.flux_attn_decode_ring(ctx, cfg, x["q"], x["cache"], x["out"])
        else:
            F.flux_kv_append(ctx, x["cache"], hkv, d, x["k_new"], x["v_new"], st["cu"], st["t"], st["max_new"])
            F.flux_attn_prefill(ctx, cfg, x["q"], st["cu"], st["max_new"], st["max_total"], x["cache"], x["mode"], x["out"])
    return {"out": [x["out"] for x in st["layers"]], "k": [x["cache"].k for x in st["layers"]], "v": [x["cache"].v for x in st["layers"]],
            "len": st["kv_len"]}


# ---- the same in float64 --------------------------------------------------------------------------------------------

def _attend(q, k, v, visible):
    """q [n, G, d], k, v [m, d] of one KV head; visible: bool, broadcast to [n, G, m].  All but `visible` in float64."""
    n, grp, d = q.shape
    s = (q.reshape(n * grp, d) @ k.t()).view(n, grp, -1).mul_(1 / math.sqrt(d))
    s.masked_fill_(~visible, -math.inf)
    p = torch.softmax(s, -1)
    return (p.view(n * grp, -1) @ v).view(n, grp, d)


def _attend_rows(case, q, k, v, pos0, fa):
    """Rows pos0 .. of one sequence and KV head, in pieces; k, v hold every position."""
    b, sink, wb = _geom(case)
    out = []
    step = max(1, 2 ** 27 // (q.shape[1] * k.shape[0]))
    for r in range(0, q.shape[0], step):
        n = min(step, q.shape[0] - r)
        i = torch.arange(pos0 + r, pos0 + r + n, device=DEV)[:, None]
        hi = pos0 + r + n
        if fa:
            at = torch.arange(hi, device=DEV)
            vis = at <= i
        else:
            lo = max(sink, _window_lo(case, pos0 + r))
            at = torch.cat([torch.arange(min(sink, hi), device=DEV), torch.arange(lo, max(lo, hi), device=DEV)])
            vis = (at <= i) & ((at < sink) | (i // b - at // b < wb))
        out.append(_attend(q[r:r + n], k[at], v[at], vis[:, None, :]))
    return torch.cat(out)


def _exact_attention(case, seed):
    if case["kind"] == "prefill":
        new, past = _ints(case["new"]), _ints(case["past"])
    else:
        past = _ints(case["lens"])
        new = [1] * len(past)
    _, sink, wb = _geom(case)
    window = wb * max(1, case["sa_block"])
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    grp = hq // hkv
    ring = case["kind"] == "ring"
    modes = _modes(case, len(new))
    outs = []
    for layer, fa in enumerate(modes):
        x = _layer_inputs(case, seed, layer, new, sink + window if ring else max(n + p for n, p in zip(new, past)) + 64)
        out = torch.zeros(sum(new), hq, d, dtype=torch.float64, device=DEV)
        at = 0
        for b, (n, p) in enumerate(zip(new, past)):
            for h in range(hkv):
                q = x["q"][at:at + n, h * grp:(h + 1) * grp].double()
                kn, vn = x["k_new"][at:at + n, h].double(), x["v_new"][at:at + n, h].double()
                if ring:                                     # stored rows, the new one in its place
                    k, v = x["k"][b, h].double(), x["v"][b, h].double()
                    r = p if p < sink else sink + (p - sink) % window
                    k[r], v[r] = kn[0], vn[0]
                    row = torch.arange(sink + window, device=DEV)
                    pos = torch.where(row < sink, row, p - (p - row) % window)         # the newest position a ring row holds
                    vis = (pos <= p) & ((row < sink) | (pos >= max(sink, _window_lo(case, p))))
                    got = _attend(q, k, v, vis[None, None])
                else:
                    k, v = torch.cat([x["k"][b, h, :p].double(), kn]), torch.cat([x["v"][b, h, :p].double(), vn])
                    got = _attend_rows(case, q, k, v, p, fa[b])
                out[at:at + n, h * grp:(h + 1) * grp] = got
            at += n
        outs.append(out)
    none = [None] * len(modes)
    return {"out": outs, "k": none, "v": none, "len": None}


def _xa_keep(q, k, n, threshold):
    """Keep matrix of one head, bool [nb, nb]: masses of 64 x 64 blocks from the antidiagonals of 16 x 16 squares."""
    d = q.shape[1]
    ns, nb = -(-n // 16), -(-n // 64)
    pad = 64 * nb - n
    q = torch.nn.functional.pad(q, (0, 0, 0, pad)).view(4 * nb, 16, d)
    k = torch.nn.functional.pad(k, (0, 0, 0, pad)).view(4 * nb, 16, d).flip(1)      # query offset r meets key offset 15 - r
    r = torch.arange(16, device=DEV)
    sq = torch.arange(4 * nb, device=DEV)
    e = q.reshape(4 * nb, -1) @ k.reshape(4 * nb, -1).t()
    q8 = (q * (r >= 8)[None, :, None]).reshape(4 * nb, -1)                           # on the diagonal only r >= 8 is causal
    e[sq, sq] = (q8 * k.reshape(4 * nb, -1)).sum(1)
    a, b = sq[:, None], sq[None, :]
    first = torch.maximum(torch.where(a == b, 8, 0), 16 * b + 16 - n).clamp(min=0)
    last = torch.clamp(n - 1 - 16 * a, max=15)
    cnt = last - first + 1
    e = torch.where((b <= a) & (cnt > 0), e / (math.sqrt(d) * cnt.clamp(min=1)), -math.inf)
    p = torch.nan_to_num(torch.softmax(e, -1))
    rows = (ns - 4 * torch.arange(nb, device=DEV)).clamp(max=4)
    mass = p.view(nb, 4, nb, 4).sum((1, 3)) / rows[:, None]
    top = mass.sort(-1, descending=True).values
    at = (top.cumsum(-1) < threshold * mass.sum(-1, keepdim=True)).sum(-1, keepdim=True).clamp(max=nb - 1)
    keep = mass >= top.gather(-1, at)
    i = torch.arange(nb, device=DEV)
    return ((keep | (i[:, None] == i)) & (i <= i[:, None]))


def _exact_xa(case, seed):
    x = _xa_inputs(case, seed)
    lens, hq, hkv, d = _ints(case["lens"]), case["hq"], case["hkv"], case["d"]
    nbm = -(-max(lens) // 64)
    keep = torch.zeros(len(lens), hq, nbm, nbm, dtype=torch.uint8, device=DEV)
    out = torch.zeros(sum(lens), hq, d, dtype=torch.float64, device=DEV)
    at = 0
    for b, n in enumerate(lens):
        nb = -(-n // 64)
        for h in range(hq):
            q, k, v = x["q"][at:at + n, h].double(), x["k_new"][at:at + n, h // (hq // hkv)].double(), x["v_new"][at:at + n, h // (hq // hkv)].double()
            kp = _xa_keep(q, k, n, case["threshold"])
            keep[b, h, :nb, :nb] = kp
            j = torch.arange(n, device=DEV)
            for r in range(0, n, 4096):
                i = torch.arange(r, min(n, r + 4096), device=DEV)
                m = int(i[-1]) + 1
                vis = (j[:m] <= i[:, None]) & kp[i // 64][:, j[:m] // 64]
                out[at + r:at + r + len(i), h] = _attend(q[i][:, None], k[:m], v[:m], vis[:, None, :])[:, 0]
        at += n
    return {"out": out, "keep": keep, "k": None, "v": None, "len": None}


def exact(case, seed):
    if case["kind"] == "router":
        x = _router_inputs(case, seed)
        w1, w2 = x["w1"].double(), x["w2"].double()
        logits, at = [], 0
        for n in _ints(case["lens"]):
            rows = x["x"][at:at + n]
            p = case["pool"]
            if p and n > 2 * p:
                rows = torch.cat([rows[:p], rows[n - p:]])
            h = w1 @ rows.double().mean(0)
            logits.append(w2 @ (h * torch.sigmoid(h)))
            at += n
        return {"logits": torch.stack(logits), "mode": None}
    return _exact_xa(case, seed) if case["kind"] == "xa" else _exact_attention(case, seed)


# ---- more cases of the same ranges ----------------------------------------------------------------------------------

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["router", "decode", "decode", "decode", "ring", "prefill", "prefill", "prefill", "prefill", "xa"])
    if kind == "router":
        return {"kind": kind, "hidden": rng.choice([2560, 3584, 4096]), "inner": rng.choice([128, 256, 512]), "pool": rng.choice([50, 100, 100]),
                "lens": _text(_log(rng, 20, 20000) for _ in range(_log(rng, 1, 8)))}
    hq, hkv, d = rng.choice([(32, 8, 128), (32, 8, 128), (28, 4, 128), (16, 8, 128), (8, 2, 64), (32, 8, 64)])
    if kind == "xa":
        return {"kind": kind, "hq": hq, "hkv": hkv, "d": d, "fp32": rng.choice([0, 0, 1]), "threshold": rng.choice([0.8, 0.9, 0.95]),
                "lens": _text(_log(rng, 1000, 20000) for _ in range(rng.choice([1, 1, 2])))}
    n_sink, window, block = rng.choice([(128, 4096, 0), (128, 4096, 64), (64, 2048, 0), (64, 2048, 64), (16, 128, 0)])
    case = {"kind": kind, "hq": hq, "hkv": hkv, "d": d, "n_sink": n_sink, "window": window, "sa_block": block, "fp32": rng.choice([0, 0, 0, 1])}
    while True:
        layers = rng.choice([1, 2, 4])
        if kind == "prefill":
            batch = _log(rng, 1, 8)
            whole = rng.random() < 0.5                       # whole prompts, or turns and chunks behind a cached context
            case["new"] = _text(_log(rng, 16, (32768 if whole else 16384) if batch == 1 else (8192 if whole else 4096)) for _ in range(batch))
            case["past"] = _text(0 if whole else _log(rng, 500, 65536) for _ in range(batch))
            layers = rng.choice([1, 1, 2])
        else:
            batch = _log(rng, 1, 32)
            longest = _log(rng, 100, 131072)
            case["lens"] = _text(_log(rng, max(1, longest // 20), longest) for _ in range(batch))
        letters = "S" if kind == "ring" else "FS"
        case["modes"] = "/".join("".join(rng.choice(letters) for _ in range(batch)) for _ in range(layers))
        w = work(case)
        rows = max(_ints(case["lens"])) if kind == "decode" else 0
        held = 4 * layers * batch * rows * hkv * d           # the caches of a decode state
        if w["flops"] <= MAX_PREFILL_FLOPS and w["bytes"] <= MAX_DECODE_BYTES and held <= 40e9:
            return case
