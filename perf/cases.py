"""Performance cases: what a program does with one attention layer's bounded cache.

Four operations, each through the package's public objects:

* ``prefill``: a new prompt goes through ``PDAttention.run_prefill`` block by
  block (attention, score sums, cut, compaction), from an empty cache;
* ``run``: the same followed by ``PDAttention.run_decode``;
* ``decode``: one generated token for every sample of the batch through the
  layers of a ``PDStack`` whose caches are full (attention, scores, one removal);
* ``long``: one token over a cache that is never cut (outputs only), as a
  program does that answers another question about a prompt it keeps.

Inputs: queries and keys N(0, 1), so logits have standard deviation 1; each
position's keys are scaled by a lognormal factor (heavy and light positions);
values N(0, 1).

Cut caches come back whole over their live entries (slots past the length are
scratch).  Cached K and V rows are copies of input rows, so they come as bit
patterns.  Where two averages at a cut lie within rounding of each other both
kept sets are correct; the shares in ``tolerance`` cover that.
"""
import math

import torch

from paper_2412_05693_amd import batchmax

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_MAX_GEN = 1 << 28      # decode goes on for as long as the program runs


def _case(op, *, name=None, dtype="bf16", b, heads, kv_heads, d=128, s, kv_max, block, steps=0,
          layers=1, rule="ave", pad_max=0, scores=True, fused_cut=True, removal=0):
    c = dict(op=op, dtype=dtype, b=b, heads=heads, kv_heads=kv_heads, d=d, s=s, kv_max=kv_max,
             block=block, steps=steps, layers=layers, rule=rule, pad_max=pad_max, scores=scores,
             fused_cut=fused_cut, removal=removal)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest use: a float32 multi-head layer, a short prompt and its answer;
        # a few dozen small calls, so latency and launches are what it costs
        _case("run", name="run-f32-mha-s512", dtype="f32", b=2, heads=4, kv_heads=4, d=64, s=512,
              kv_max=128, block=64, steps=32),
        # one user's prompt (time to first token): eight KV heads are all the units there are
        _case("prefill", name="prefill-b1-s4096", b=1, heads=32, kv_heads=8, s=4096, kv_max=512,
              block=256),
        # an ordinary batch through one layer of an 8B model's shape
        _case("prefill", name="prefill-b64-s4096", b=64, heads=32, kv_heads=8, s=4096, kv_max=512,
              block=256),
        # long documents, a larger cache and block
        _case("prefill", name="prefill-b32-s16384", b=32, heads=32, kv_heads=8, s=16384,
              kv_max=1024, block=512),
        # throughput serving: short prompts, a large batch
        _case("prefill", name="prefill-b256-s2048", b=256, heads=32, kv_heads=8, s=2048,
              kv_max=512, block=256),
        # the 13B multi-head shape with prompts of different lengths, padded on the left
        _case("prefill", name="prefill-mha-padded-s3584", b=8, heads=40, kv_heads=40, s=3584,
              kv_max=1024, block=256, pad_max=1024),
        # small heads, two queries per KV head, odd sizes, ranked by the last query's
        # weights, blocks and cuts as calls of their own
        _case("prefill", name="prefill-d64-tova-s1999", b=5, heads=16, kv_heads=8, d=64, s=1999,
              kv_max=333, block=100, rule="tova", fused_cut=False),
        # decoding-only compression keeps the whole prompt: attention outputs alone
        _case("prefill", name="prefill-full-s8192", b=4, heads=32, kv_heads=8, s=8192, kv_max=8192,
              block=256, scores=False),
        # one user's next token through some of a model's layers
        _case("decode", name="decode-b1", b=1, heads=32, kv_heads=8, s=4096, kv_max=512, block=256,
              layers=8),
        # an ordinary batch's next token
        _case("decode", name="decode-b64", b=64, heads=32, kv_heads=8, s=4096, kv_max=512,
              block=256, layers=4),
        # throughput serving: the largest decode batch
        _case("decode", name="decode-b1024", b=1024, heads=32, kv_heads=8, s=2048, kv_max=512,
              block=256),
        # a token over a whole 8192-token prompt, nothing removed
        _case("long", name="long-b8-n8192", b=8, heads=32, kv_heads=8, s=8192, kv_max=8448,
              block=256, scores=False),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.random()
    while True:
        d = rng.choice((64, 128, 128))
        group = rng.choice((1, 2, 4, 4))
        kv_heads = rng.choice((1, 2, 4, 5, 8, 8))
        dtype = rng.choice(("bf16",) * 7 + ("f32",))
        rule = rng.choice(("ave",) * 5 + ("sum", "recent", "tova"))
        shape = dict(dtype=dtype, heads=kv_heads * group, kv_heads=kv_heads, d=d, rule=rule)
        if kind < 0.55:
            s = _log_int(rng, 256, 16384)
            case = _case("prefill", b=_log_int(rng, 1, 256), s=s, kv_max=_log_int(rng, 64, 2048),
                         block=rng.choice((64, 128, 256, 512, _log_int(rng, 33, 512))),
                         fused_cut=rng.random() < 0.8,
                         pad_max=rng.choice((0, 0, 0, s // 3)), **shape)
            if rng.random() < 0.15:      # the whole prompt kept, outputs alone
                case.update(kv_max=s, rule="recent", scores=False, pad_max=0)
        elif kind < 0.63:
            case = _case("run", b=_log_int(rng, 1, 16), s=_log_int(rng, 128, 2048),
                         kv_max=_log_int(rng, 32, 512), block=rng.choice((32, 64, 128, 100)),
                         steps=rng.randint(8, 32), **shape)
        elif kind < 0.92:
            kv = _log_int(rng, 64, 4096)
            case = _case("decode", b=_log_int(rng, 1, 1024), s=kv + _log_int(rng, 64, 8192),
                         kv_max=kv, block=256, layers=rng.choice((1, 2, 4, 8)),
                         removal=rng.choice((0, 0, 0, min(kv, 32))), **shape)
            if rule == "tova":           # its weights live in the workspace the layers share
                case["removal"] = 0
        else:
            n = _log_int(rng, 4200, 32768)
            shape["rule"] = "recent"
            case = _case("long", b=_log_int(rng, 1, 32), s=n, kv_max=n + 64, block=256,
                         scores=False, **shape)
        w = work(case)
        slow = 16 if dtype == "f32" else 1          # float32 matrix instructions' rate
        state = w["bytes"] + 8 * case["b"] * kv_heads * (case["kv_max"] + 512) * d * case["layers"]
        calls = case["layers"] + case["s"] // case["block"] * (case["op"] in ("prefill", "run"))
        if w["flops"] * slow < 6e12 and w["bytes"] < 2.5e9 * (4 if case["op"] == "prefill" else 1) \
                and state < 2e10 and calls < 300:
            return case


def _rows_seen(case):
    """(query, visible key) pairs of one query head over the prompt, padding aside."""
    total = length = 0
    for t0 in range(0, case["s"], case["block"]):
        n = min(case["block"], case["s"] - t0)
        total += n * length + n * (n + 1) // 2
        length = min(case["kv_max"], length + n)
    return total


def work(case):
    """Every input read once, every output written once; 4 d flops per visible
    (query, key) pair (two contractions).  Padded prompts count as unpadded."""
    b, h, hk, d = case["b"], case["heads"], case["kv_heads"], case["d"]
    es = 2 if case["dtype"] == "bf16" else 4
    entry = 2 * d * es + 8                     # a cached pair, its score and position
    byts = flops = 0
    if case["op"] in ("prefill", "run"):
        kept = min(case["s"], case["kv_max"])
        byts += b * case["s"] * (2 * h + 2 * hk) * d * es + b * hk * kept * entry
        flops += 4 * d * b * h * _rows_seen(case)
    if case["op"] == "run":
        n = min(case["s"], case["kv_max"])
        byts += case["steps"] * b * (2 * h + 2 * hk) * d * es
        flops += case["steps"] * 4 * d * b * h * (n + 1)
    if case["op"] in ("decode", "long"):
        n = case["kv_max"] if case["op"] == "decode" else case["s"]
        step = b * (2 * h + 2 * hk) * d * es + b * hk * (n * 2 * d * es + entry)
        if case["op"] == "decode":             # scores read and written, positions read
            step += b * hk * n * 12
        byts += case["layers"] * step
        flops += case["layers"] * 4 * d * b * h * (n + 1)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """bf16: outputs are rounded to 8 bits (2e-3 measured against 64-bit sums).
    float32: sums of up to a few thousand terms (4e-7 to 1e-6 measured).  ``max`` and
    ``differ`` leave room for a cut between averages that rounding cannot part:
    it exchanges one light entry of one unit, and compaction then pairs the
    holes behind it with other survivors."""
    if case["dtype"] == "bf16":
        return {"rel": 0.01, "max": 0.5, "differ": 0.002}
    return {"rel": 4e-6, "max": 0.01, "differ": 0.002}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, dt):
    return torch.randn(shape, generator=g, device="cuda", dtype=dt)


def _keys(g, shape, dt):
    """N(0, 1) rows times a lognormal factor per (sample, head, position)."""
    k = _normal(g, shape, dt)
    f = torch.exp(0.5 * torch.randn(shape[:3] + (1,), generator=g, device="cuda"))
    return k.mul_(f.to(dt))


def _pads(case, g):
    pads = torch.randint(0, case["pad_max"] + 1, (case["b"],), generator=g, device="cuda",
                         dtype=torch.int32)
    pads[0] = 0
    return pads


def _prompt(case, seed):
    g, dt = _generator(seed), _DTYPES[case["dtype"]]
    b, h, hk, d = case["b"], case["heads"], case["kv_heads"], case["d"]
    t = case["s"] + case["steps"]
    x = {"q": _normal(g, (b, h, t, d), dt), "k": _keys(g, (b, hk, t, d), dt),
         "v": _normal(g, (b, hk, t, d), dt)}
    x["pads"] = _pads(case, g) if case["pad_max"] else None
    return x


def _full_cache(case, g):
    """One layer's state after a prompt: kv_max entries in each unit, scores as
    averages (light and heavy entries) times the number of queries seen."""
    b, hk, d, n, s = case["b"], case["kv_heads"], case["d"], case["kv_max"], case["s"]
    dt = _DTYPES[case["dtype"]]
    x = {"ck": _keys(g, (b, hk, n, d), dt), "cv": _normal(g, (b, hk, n, d), dt)}
    if case["op"] == "long":
        x["ck"], x["cv"] = x["ck"][:, :, :s].contiguous(), x["cv"][:, :, :s].contiguous()
        x["pos"] = torch.arange(s, device="cuda", dtype=torch.int32).expand(b, hk, s).contiguous()
        x["score"] = torch.zeros((b, hk, s), device="cuda")
        return x
    # n increasing positions below s: one in each of n equal segments
    seg = s / n
    u = torch.rand((b, hk, n), generator=g, device="cuda")
    i = torch.arange(n, device="cuda")
    lo, hi = torch.floor(i * seg), torch.floor((i + 1) * seg)
    x["pos"] = torch.minimum(lo + torch.floor(u * (hi - lo)), hi - 1).to(torch.int32)
    group = case["heads"] // hk
    ave = torch.exp(0.5 * torch.randn((b, hk, n), generator=g, device="cuda")) * group / (n + 1)
    x["score"] = ave * (s - x["pos"])
    return x


def _step(case, g):
    b, h, hk, d, dt = case["b"], case["heads"], case["kv_heads"], case["d"], _DTYPES[case["dtype"]]
    return {"q": _normal(g, (b, h, 1, d), dt), "k": _keys(g, (b, hk, 1, d), dt),
            "v": _normal(g, (b, hk, 1, d), dt)}


def _layers(case, seed):
    g = _generator(seed)
    return [(_full_cache(case, g), _step(case, g)) for _ in range(case["layers"])]


def _shape(case):
    return dict(b=case["b"], s=case["s"], kv_max=case["kv_max"], block=case["block"],
                n_heads=case["heads"], n_kv_heads=case["kv_heads"], head_dim=case["d"],
                dtype=case["dtype"])


def _set_options(att, case):
    if case["rule"] != "ave":
        att.set_rank_rule(case["rule"])
    if not case["scores"]:
        att.set_score_accumulation(False)
    if case["removal"]:
        att.set_decode_removal(case["removal"])


def prepare(case, seed):
    if case["op"] in ("prefill", "run"):
        x = _prompt(case, seed)
        att = batchmax.PDAttention(max_gen=case["steps"], **_shape(case))
        _set_options(att, case)
        if x["pads"] is not None:
            att.set_left_padding(x["pads"])
        return {"case": case, "att": att, "o": torch.empty_like(x["q"]), **x}
    stack = batchmax.PDStack(n_layers=case["layers"], max_gen=_MAX_GEN, **_shape(case))
    rows = []
    for att, (cache, row) in zip(stack.layers, _layers(case, seed)):
        n = cache["pos"].shape[2]
        att.k[:, :, :n], att.v[:, :, :n] = cache["ck"], cache["cv"]
        att.pos[:, :, :n], att.score[:, :, :n] = cache["pos"], cache["score"]
        att.len.fill_(n)
        _set_options(att, case)
        att.resume(n, case["s"])
        row["o"] = torch.empty_like(row["q"])
        rows.append(row)
    return {"case": case, "stack": stack, "rows": rows, "pos": case["s"]}


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def _bits(x):
    return x.view(torch.int16 if x.dtype == torch.bfloat16 else torch.int32)


def _live(att):
    n = att.length
    return {"k": _bits(att.k)[:, :, :n], "v": _bits(att.v)[:, :, :n], "score": att.score[:, :, :n],
            "pos": att.pos[:, :, :n], "len": att.len}


def run(state):
    case = state["case"]
    if case["op"] in ("prefill", "run"):
        att, q, k, v, o = (state[x] for x in ("att", "q", "k", "v", "o"))
        att.reset()
        att.run_prefill(q, k, v, o, fused_cut=case["fused_cut"])
        if case["op"] == "run":
            att.run_decode(q, k, v, o)
        return {"o": o, **_live(att)}
    if case["op"] == "decode":
        pos = state["pos"]
        for att, r in zip(state["stack"].layers, state["rows"]):
            att.decode_step(pos, r["q"], r["k"], r["v"], r["o"])
        state["pos"] = pos + 1
    else:
        # back to the prompt's end: the kept prompt takes the next question's token
        for att, r in zip(state["stack"].layers, state["rows"]):
            att.resume(case["s"], case["s"])
            att.decode_step(case["s"], r["q"], r["k"], r["v"], r["o"])
    return [{"o": r["o"], **_live(att)} for att, r in zip(state["stack"].layers, state["rows"])]


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
_NEG = float("-inf")


def _attend(q, kk, vv, hidden, scale):
    """q [u, G, n, d], kk/vv [u, L, d], hidden [u, n, L] -> o, probabilities."""
    u, g, n, d = q.shape
    z = torch.bmm(q.reshape(u, g * n, d), kk.transpose(1, 2).contiguous()).view(u, g, n, -1) * scale
    z.masked_fill_(hidden[:, None], _NEG)
    m = z.amax(dim=-1, keepdim=True)
    m = torch.where(torch.isinf(m), torch.zeros_like(m), m)
    p = torch.exp(z - m)
    p /= p.sum(dim=-1, keepdim=True).clamp_min(1e-300)
    o = torch.bmm(p.view(u, g * n, -1), vv).view(u, g, n, d)
    return o, p


def _cut(st, keep, curr, rule):
    """Keep `keep` entries: remove the smallest (key, position), then fill the
    holes below `keep` with the survivors above it, both in slot order."""
    n = st["pos"].shape[1]
    pos = st["pos"].double()
    key = {"ave": lambda: st["score"] / (curr + 1 - pos), "sum": lambda: st["score"],
           "recent": lambda: pos, "tova": lambda: st["last"]}[rule]()
    by_pos = torch.argsort(pos, dim=1, stable=True)
    order = by_pos.gather(1, torch.argsort(key.gather(1, by_pos), dim=1, stable=True))
    gone = torch.zeros_like(key, dtype=torch.bool).scatter_(1, order[:, :n - keep], True)
    hole = gone[:, :keep]
    slots = torch.arange(keep, n, device=pos.device).expand(pos.shape[0], -1)
    src = torch.sort(torch.where(gone[:, keep:], n, slots), dim=1).values
    idx = torch.arange(keep, device=pos.device).expand(pos.shape[0], -1)
    if n > keep:
        rank = (torch.cumsum(hole.long(), dim=1) - 1).clamp(0, n - keep - 1)
        idx = torch.where(hole, src.gather(1, rank).clamp_max(n - 1), idx)
    for name in ("score", "pos", "last"):
        st[name] = st[name].gather(1, idx)
    for name in ("k", "v"):
        st[name] = st[name].gather(1, idx[..., None].expand(-1, -1, st[name].shape[2]))


def _append(st, k, v, t0):
    u, n = k.shape[:2]
    zero = torch.zeros((u, n), device="cuda", dtype=torch.float64)
    t = torch.arange(t0, t0 + n, device="cuda").expand(u, n)
    for name, x in (("k", k), ("v", v), ("score", zero), ("last", zero), ("pos", t)):
        st[name] = torch.cat([st[name], x], dim=1)


def _decode_exact(case, st, q, k, v, pos):
    """One step of the units in `st`; q [u, G, 1, d], k and v [u, 1, d]."""
    n, keep, rule = st["pos"].shape[1], case["kv_max"], case["rule"]
    if case["removal"] and n >= keep:
        _cut(st, keep - case["removal"], pos - 1, rule)
    _append(st, k, v, pos)
    hidden = torch.zeros((q.shape[0], 1, st["pos"].shape[1]), device="cuda", dtype=torch.bool)
    if st["pad"] is not None:
        hidden = st["pos"][:, None] < st["pad"][:, None, None]
    o, p = _attend(q, st["k"], st["v"], hidden, 1.0 / math.sqrt(case["d"]))
    st["last"] = p.sum(dim=(1, 2))
    if case["op"] != "long":
        st["score"] = st["score"] + st["last"]
        if st["pos"].shape[1] > keep:
            _cut(st, keep, pos, rule)
    return o


def _prefill_exact(case, st, q, k, v, o):
    s, rule = case["s"], case["rule"]
    for t0 in range(0, s, case["block"]):
        t1 = min(s, t0 + case["block"])
        n = t1 - t0
        _append(st, k[:, t0:t1], v[:, t0:t1], t0)
        rows = torch.arange(t0, t1, device="cuda")
        hidden = st["pos"][:, None, :] > rows[None, :, None]
        if st["pad"] is not None:
            pad = st["pad"][:, None, None]
            hidden = hidden | (st["pos"][:, None, :] < pad) | (rows[None, :, None] < pad)
        o[:, :, t0:t1], p = _attend(q[:, :, t0:t1], st["k"], st["v"], hidden,
                                    1.0 / math.sqrt(case["d"]))
        if case["scores"]:
            st["score"] = st["score"] + p.sum(dim=(1, 2))
            st["last"] = p[:, :, n - 1].sum(dim=1)
        if st["pos"].shape[1] > case["kv_max"]:
            _cut(st, case["kv_max"], t1 - 1, rule)


def _chunks(case, rows, length):
    """Units at a time, so that the logits of a chunk stay near 1 GB."""
    group = case["heads"] // case["kv_heads"]
    units = case["b"] * case["kv_heads"]
    n = max(1, min(units, int(1.2e8 / (group * rows * length))))
    return [(u, min(units, u + n)) for u in range(0, units, n)]


def exact(case, seed):
    """Outputs, and scores where so few cuts are made that kept sets hardly ever
    hang on rounding; positions and rows (copies) are not computed numbers."""
    b, h, hk, d = case["b"], case["heads"], case["kv_heads"], case["d"]
    units, group = b * hk, h // hk
    if case["op"] in ("prefill", "run"):
        x = _prompt(case, seed)
        t = case["s"] + case["steps"]
        cuts = max(0, (case["s"] - case["kv_max"])) // case["block"] + case["steps"]
        o = torch.empty((units, group, t, d), device="cuda", dtype=torch.float64)
        scores = []
        for u0, u1 in _chunks(case, case["block"], case["kv_max"] + case["block"]):
            q = x["q"].view(units, group, t, d)[u0:u1].double()
            k, v = (x[y].view(units, t, d)[u0:u1].double() for y in ("k", "v"))
            empty = torch.zeros((u1 - u0, 0), device="cuda", dtype=torch.float64)
            st = {"k": k[:, :0], "v": v[:, :0], "score": empty, "last": empty,
                  "pos": empty.long(), "pad": None}
            if x["pads"] is not None:
                st["pad"] = x["pads"].long().repeat_interleave(hk)[u0:u1]
            _prefill_exact(case, st, q, k, v, o[u0:u1])
            for i in range(case["steps"]):
                r = case["s"] + i
                o[u0:u1, :, r:r + 1] = _decode_exact(case, st, q[:, :, r:r + 1], k[:, r:r + 1],
                                                     v[:, r:r + 1], r)
            scores.append(st["score"])
        score = torch.cat(scores).view(b, hk, -1) if units * cuts <= 400 else None
        return {"o": o.view(b, h, t, d), "k": None, "v": None, "score": score, "pos": None,
                "len": None}
    out = []
    for cache, row in _layers(case, seed):
        os_, scores = [], []
        for u0, u1 in _chunks(case, 1, (case["kv_max"] + 1) * d):
            def unit(y, n, dt=torch.float64):
                return y.view((units, n) + tuple(y.shape[3:]))[u0:u1].to(dt)
            n = cache["pos"].shape[2]
            st = {"k": unit(cache["ck"], n), "v": unit(cache["cv"], n),
                  "score": unit(cache["score"], n), "pos": unit(cache["pos"], n, torch.long),
                  "pad": None}
            st["last"] = torch.zeros_like(st["score"])
            q = row["q"].view(units, group, 1, d)[u0:u1].double()
            os_.append(_decode_exact(case, st, q, unit(row["k"], 1), unit(row["v"], 1), case["s"]))
            scores.append(st["score"])
        few = units * case["layers"] <= 400 and not case["removal"]
        out.append({"o": torch.cat(os_).view(b, h, 1, d), "k": None, "v": None,
                    "score": torch.cat(scores).view(b, hk, -1) if few else None, "pos": None,
                    "len": None})
    return out
