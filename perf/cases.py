"""Performance cases: the calls that a decoder makes of this library, through its public binding.

A case is a dict of plain values.  Its kind says which calls one pass makes on which cache:

* ``refresh``: one decode step that scores, folds and evicts (KvCache / evict_step) on a cache at its budget;
* ``stale``: one decode step between refreshes (Lazy, Score-Free): prior, eviction on the stale ranking, append;
* ``decode``: one decode step around the model's own attention: kv_append, kv_attend_score layer by layer with
  the score emitted, kv_evict_finish;
* ``score``: the first step's scoring and selection over a whole prefill (kv_score_ema, kv_topk_select);
* ``compact``: the first step's compaction of that prefill to the budget (kv_compact).

A pass advances the state as a decode loop does: the next pass is the next step, with the next position and the
next of a few prepared step inputs.  ``context`` is the prefill length (it sets the cache's capacity, as in a
program that prefills and then decodes in place), ``budget`` the tokens kept.
"""
import math

import torch

from paper_2609_03515_amd import binding as B

STEPS = 8  # prepared step inputs (queries and newcomers), taken in turn


def _case(name, kind, batch, layers, hq, hkv, d, dtype, context, budget, **more):
    c = {"name": name, "kind": kind, "batch": batch, "layers": layers, "hq": hq, "hkv": hkv, "d": d, "dtype": dtype,
         "context": context, "budget": budget, "alpha": 0.9, "window": 64}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: a two-layer float32 cache of 51 tokens; launches and host work are all there is
        _case("tiny_refresh", "refresh", 1, 2, 4, 2, 64, "f32", 512, 51, window=0),
        # the benchmark's step: 8B-shaped decoder at 32k context, 10% of the tokens kept
        _case("llama8b_refresh", "refresh", 8, 32, 32, 8, 128, "bf16", 32768, 3277),
        # the same decoder serving one sequence (latency)
        _case("llama8b_refresh_b1", "refresh", 1, 32, 32, 8, 128, "bf16", 32768, 3277),
        # a decoder with 7 query heads per KV head and a large batch at a short context
        _case("qwen7b_refresh", "refresh", 32, 28, 28, 4, 128, "bf16", 8192, 2048, alpha=0.8, window=0),
        # the value-norm scorer with its norm cache
        _case("llama8b_refresh_vnorm", "refresh", 8, 32, 32, 8, 128, "bf16", 32768, 3277, variant="vnorm"),
        # Lazy refresh: three of four steps are these (mean prior)
        _case("llama8b_stale", "stale", 8, 32, 32, 8, 128, "bf16", 32768, 3277, prior="mean"),
        # Score-Free decoding of a 128k context (lowest prior): every step after the first
        _case("scorefree_stale", "stale", 2, 32, 32, 8, 128, "bf16", 131072, 13107, prior="min"),
        # decoder-order attention with the score emitted, and the eviction that ends the step
        _case("llama8b_decode", "decode", 8, 32, 32, 8, 128, "bf16", 32768, 3277),
        _case("llama8b_decode_b1", "decode", 1, 32, 32, 8, 128, "bf16", 32768, 3277),
        _case("qwen7b_decode", "decode", 32, 28, 28, 4, 128, "bf16", 8192, 2048, alpha=0.8, window=0),
        # the first step over the 32k prefill: every token scored and the kept ones chosen, ...
        _case("llama8b_prefill_score", "score", 8, 32, 32, 8, 128, "bf16", 32768, 3277),
        # ... and their rows moved together
        _case("llama8b_prefill_compact", "compact", 8, 32, 32, 8, 128, "bf16", 32768, 3277),
    ]


# Head layouts drawn from: the two decoders above, and the group sizes and widths that the tests run.
_HEADS = ((32, 8, 128), (32, 8, 128), (28, 4, 128), (28, 4, 128), (40, 8, 128), (16, 8, 64), (32, 4, 128), (4, 2, 64))
_ROWS = 3277 * 32 * 8 * 8  # K rows that a steady step of the largest listed case reads


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("refresh", "refresh", "stale", "decode", "decode", "score", "compact"))
    while True:
        hq, hkv, d = rng.choice(_HEADS)
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        batch, layers = log_int(1, 32), log_int(2, 32)
        context = log_int(512, 131072)
        budget = max(16, int(context * rng.uniform(0.08, 0.3)))
        width = d * (4 if dtype == "f32" else 2) / 256.0
        slabs = batch * layers * hkv
        rows = context if kind in ("score", "compact") else budget
        most = 9 * _ROWS if kind in ("score", "compact") else _ROWS  # no more work than the listed ones
        if slabs * rows * width <= most and slabs * context * width <= 9 * _ROWS:
            break
    c = _case("", kind, batch, layers, hq, hkv, d, dtype, context, budget)
    del c["name"]
    c["alpha"] = rng.choice((0.8, 0.9))
    c["window"] = rng.choice((0, 64))
    if kind == "refresh":
        c["variant"] = rng.choice(("plain", "plain", "vnorm", "entropy"))
    if kind == "stale":
        c["prior"] = rng.choice(("mean", "min"))
    return c


# ---- inputs -------------------------------------------------------------------------------------------------
# Keys, queries and values ~ N(0, 1); 2% of the tokens are heavy hitters whose keys lean towards a direction that
# every query of the KV head shares (expected logit raised by 3), as attention sinks and topic tokens do.

def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1_000_003 + tag * 7919 + 12345) % (1 << 62))
    return g


def _draws(case, seed, values):
    """k, v (None unless `values`), pos, u: the cache before the first pass, and the step inputs."""
    L, b, hq, hkv, d = (case[x] for x in ("layers", "batch", "hq", "hkv", "d"))
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    cap = case["context"] + 1
    prefill = case["kind"] in ("score", "compact")
    n = cap if prefill else case["budget"]
    dev = "cuda"
    dirs = torch.randn(L, hkv, d, generator=_gen(seed, 0), device=dev)
    dirs = dirs / dirs.norm(dim=-1, keepdim=True) * d ** 0.25
    heavy = torch.rand(b, n, generator=_gen(seed, 1), device=dev) < 0.02
    k = torch.empty(L, b, hkv, cap, d, dtype=dt, device=dev)
    v = torch.empty_like(k) if values else None
    gk, gv = _gen(seed, 2), _gen(seed, 3)
    lean = (3.0 * heavy)[:, None, :, None].to(dt)
    for l in range(L):
        if n < cap:
            k[l, :, :, n:].zero_()
        k[l, :, :, :n].normal_(generator=gk)
        k[l, :, :, :n] += lean * dirs[l][None, :, None, :].to(dt)
        if v is not None:
            if n < cap:
                v[l, :, :, n:].zero_()
            v[l, :, :, :n].normal_(generator=gv)
    pos = torch.zeros(b, cap, dtype=torch.int32, device=dev)
    u = torch.zeros(b, cap, dtype=torch.float32, device=dev)
    if prefill:
        pos[:] = torch.arange(cap, dtype=torch.int32, device=dev)
    else:  # a cache in the middle of decoding: a subset of the context, the newest token in it
        pick = torch.rand(b, case["context"] - 1, generator=_gen(seed, 4), device=dev).topk(n - 1, dim=1).indices
        pos[:, : n - 1] = pick.sort(dim=1).values.to(torch.int32)
        pos[:, n - 1] = case["context"] - 1
        uu = torch.randn(b, n, generator=_gen(seed, 5), device=dev).exp()
        u[:, :n] = uu / uu.sum(dim=1, keepdim=True)
    steps, gs = [], _gen(seed, 6)
    for _ in range(1 if case["kind"] == "compact" else STEPS):
        q = torch.randn(L, b, hq, d, generator=gs, device=dev) + dirs.repeat_interleave(hq // hkv, dim=1)[:, None]
        kn = torch.randn(L, b, hkv, d, generator=gs, device=dev)
        vn = torch.randn(L, b, hkv, d, generator=gs, device=dev)
        steps.append((q.to(dt), kn.to(dt), vn.to(dt)))
    keep = None
    if case["kind"] == "compact":  # B kept tokens anywhere in the prefill, the newest among them
        keep = torch.zeros(b, cap, dtype=torch.uint8, device=dev)
        pick = torch.rand(b, cap - 1, generator=_gen(seed, 7), device=dev).topk(case["budget"] - 1, dim=1).indices
        keep.scatter_(1, pick, 1)
        keep[:, cap - 1] = 1
        u = torch.rand(b, cap, generator=_gen(seed, 8), device=dev)
    return k, v, pos, u, steps, keep


def _bias(case):
    return (0.5 if case["window"] else 0.0), case["window"]


def prepare(case, seed):
    kind = case["kind"]
    k, v, pos, u, steps, keep = _draws(case, seed, kind != "score")
    cap = case["context"] + 1
    shape = B.make_shape(case["batch"], case["layers"], case["hq"], case["hkv"], case["d"], cap, case["dtype"])
    bias, window = _bias(case)
    variant = case.get("variant", "plain")
    params = B.make_params(case["alpha"], case["budget"], score_free=kind == "stale",
                           nonrefresh_init=case.get("prior", "mean"), recency_bias=bias, recency_window=window,
                           vnorm=variant == "vnorm", entropy=variant == "entropy")
    s = {"kind": kind, "shape": shape, "params": params, "steps": steps, "t": 2, "new_pos": case["context"],
         "n": cap if kind in ("score", "compact") else case["budget"], "budget": case["budget"],
         "bias": bias, "window": window, "alpha": case["alpha"]}
    if kind in ("refresh", "stale"):
        norms = None
        if variant == "vnorm":
            norms = torch.zeros(case["layers"], case["batch"], case["hkv"], cap, dtype=torch.float32, device="cuda")
            B.kv_value_norms(shape, case["budget"], v, norms)
        # the scratch of a steady step, not of the first one: a decoder that prefills elsewhere allocates this
        s["cache"] = B.KvCache(shape, k, v, u, pos, case["budget"], B.workspace(shape, case["budget"] + 1), norms)
    else:
        s.update(k=k, v=v, u=u, pos=pos, keep=keep, ws=B.workspace(shape, s["n"] + (kind == "decode")))
    if kind == "score":
        s["keep"] = torch.zeros(case["batch"], cap, dtype=torch.uint8, device="cuda")
    if kind == "decode":  # the per-layer tensors that a model's layers hold
        s["o"] = torch.zeros(case["layers"], case["batch"], case["hq"], case["d"], dtype=k.dtype, device="cuda")
        s["layers"] = [[(q[l], s["o"][l]) for l in range(case["layers"])] for q, _, _ in steps]
    return s


def run(s):
    kind, t, new_pos = s["kind"], s["t"], s["new_pos"]
    i = (t - 2) % len(s["steps"])
    q, k_new, v_new = s["steps"][i]
    s["t"], s["new_pos"] = t + 1, new_pos + 1
    if kind in ("refresh", "stale"):
        c = s["cache"]
        n = B.evict_step(c, q, k_new, v_new, t, s["params"], new_pos)
        out = {"k": c.k[:, :, :, :n], "v": c.v[:, :, :, :n], "u": c.u[:, :n], "pos": c.pos[:, :n]}
        if c.v_norms is not None:
            out["norms"] = c.v_norms[:, :, :, :n]
        return out
    shape, k, v, u, pos, ws, n = s["shape"], s["k"], s["v"], s["u"], s["pos"], s["ws"], s["n"]
    if kind == "decode":
        B.kv_append(shape, s["params"], t, n, new_pos, k_new, v_new, k, v, u, pos)
        for l, (ql, ol) in enumerate(s["layers"][i]):
            B.kv_attend_score(shape, l, 1, n + 1, ql, k, v, pos, new_pos, s["bias"], s["window"], B.KV_EMIT_SCORES,
                              ol, ws)
        n = B.kv_evict_finish(shape, s["params"], t, n + 1, k, v, u, pos, ws)
        return {"o": s["o"], "k": k[:, :, :, :n], "v": v[:, :, :, :n], "u": u[:, :n], "pos": pos[:, :n]}
    if kind == "score":  # the prefill's last token (position n - 1) asks
        B.kv_score_ema(shape, n, q, k, pos, n - 1, s["alpha"], s["bias"], s["window"], u, None, ws)
        B.kv_topk_select(shape, n, s["budget"], u, pos, s["keep"], ws)
        return {"u": u, "keep": s["keep"]}
    # compact: the same decision again moves the same rows again
    B.kv_compact(shape, n, s["budget"], s["keep"], k, v, u, pos, ws)
    m = s["budget"]
    return {"k": k[:, :, :, :m], "v": v[:, :, :, :m], "u": u[:, :m], "pos": pos[:, :m]}


# ---- what a pass cannot do without ---------------------------------------------------------------------------

def work(case):
    L, b, hq, hkv, d = (case[x] for x in ("layers", "batch", "hq", "hkv", "d"))
    e = 4 if case["dtype"] == "f32" else 2
    slabs, heads, m = L * b * hkv, L * b * hq, case["budget"]
    row, n_all = d * e, case["context"] + 1
    newcomer = 4 * slabs * row  # its K and V rows read and written
    if case["kind"] == "refresh":
        n = m + 1
        norms = 4 * slabs * n if case.get("variant") == "vnorm" else 0
        return {"bytes": slabs * m * row + heads * row + newcomer + norms + b * n * 12, "flops": 2 * heads * n * d}
    if case["kind"] == "stale":
        return {"bytes": newcomer + b * m * 8, "flops": 2 * b * m}
    if case["kind"] == "decode":
        n = m + 1
        return {"bytes": 2 * slabs * m * row + 2 * heads * row + newcomer + b * n * 12, "flops": 4 * heads * n * d}
    if case["kind"] == "score":
        return {"bytes": slabs * n_all * row + heads * row + b * n_all * 13, "flops": 2 * heads * n_all * d}
    moved = b * m * (1.0 - m / n_all)  # kept tokens above the budget's rows, on average
    return {"bytes": 4 * L * hkv * row * moved + b * n_all, "flops": 0}


def tolerance(case):
    # Utilities are float32 sums of exponentials: 6e-8 to 8e-8 from the 64-bit value as measured, and as much from
    # one order of the sums to another.  Rows, positions and decisions are copies that those sums decide (the
    # neighbour of an evicted utility lies a relative 1e-4 away; of 32k utilities cut at the budget a few may tie).
    kind, f32 = case["kind"], case["dtype"] == "f32"
    if kind == "compact":
        return "exact"
    if kind == "stale":
        return {"rel": 2e-6, "max": 1e-4, "differ": 0.0}
    if kind == "score":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-4}
    if kind == "refresh" or f32:
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    # the attention output is rounded to bf16: sums that differ by 1e-7 round apart once in some ten thousand
    # (2.9e-5 measured between two runs, whose waves add their blocks in another order)
    return {"rel": 2e-4, "max": 1.6e-2, "differ": 0.0}


# ---- the same in 64 bits -------------------------------------------------------------------------------------

def _attention(case, k, q, pos, cur_pos, l):
    """[b, hkv, group, n] attention of layer l's query heads over the rows of k[l] (float64)."""
    b, hq, hkv, d = (case[x] for x in ("batch", "hq", "hkv", "d"))
    n = k.shape[3]
    qd = q[l].double().reshape(b * hkv, hq // hkv, d).transpose(1, 2).contiguous()
    z = torch.bmm(k[l].double().reshape(b * hkv, n, d), qd).reshape(b, hkv, n, hq // hkv) / math.sqrt(d)
    bias, window = _bias(case)
    if window:
        z += (bias * (pos >= cur_pos - (window - 1)).double())[:, None, :, None]
    return torch.softmax(z, dim=2).transpose(2, 3)


def exact(case, seed):
    kind = case["kind"]
    k, v, pos, u, steps, keep = _draws(case, seed, kind != "score")
    L, b, hq, hkv, m = case["layers"], case["batch"], case["hq"], case["hkv"], case["budget"]
    q, k_new, v_new = steps[0]
    ud, alpha = u.double(), case["alpha"]
    if kind == "compact":
        for s in range(b):
            hole = (keep[s, :m] == 0).nonzero()[:, 0]
            tail = (keep[s, m:] != 0).nonzero()[:, 0] + m
            for x in (k, v):
                x[:, s][:, :, hole] = x[:, s][:, :, tail]
            u[s, hole] = u[s, tail]
            pos[s, hole] = pos[s, tail]
        return {"k": k[:, :, :, :m].double(), "v": v[:, :, :, :m].double(), "u": u[:, :m].double(), "pos": pos[:, :m]}
    cur = case["context"]
    if kind == "score":
        for l in range(L):
            ud = alpha * ud + (1.0 - alpha) * _attention(case, k, q, pos, cur, l).sum(dim=(1, 2)) / hq
        return {"u": ud, "keep": None}
    n = m + 1  # the newcomer is row n - 1
    k, v, pos, ud = k[:, :, :, :n], v[:, :, :, :n], pos[:, :n], ud[:, :n].clone()
    k[:, :, :, m], v[:, :, :, m], pos[:, m] = k_new, v_new, cur
    o = []
    if kind == "stale":
        ud[:, m] = ud[:, :m].mean(dim=1) if case["prior"] == "mean" else ud[:, :m].min(dim=1).values
    else:
        ud[:, m] = 0.0
        variant = case.get("variant", "plain")
        for l in range(L):
            a = _attention(case, k, q, pos, cur, l)
            if kind == "decode":
                vd = v[l].double().reshape(b * hkv, n, -1)
                o.append(torch.bmm(a.reshape(b * hkv, hq // hkv, n).contiguous(), vd).reshape(b, hq, -1))
            s = a.sum(dim=(1, 2)) / hq
            if variant == "entropy":
                s = s * (-(s * s.log()).sum(dim=1) / math.log(n))[:, None]
            if variant == "vnorm":
                vn = v[l].double().norm(dim=-1)
                s = (a * (vn / vn.mean(dim=-1, keepdim=True))[:, :, None]).sum(dim=(1, 2)) / hq
            ud = alpha * ud + (1.0 - alpha) * s
    for s in range(b):  # the lowest utility leaves, the highest position among equals
        low = (ud[s] == ud[s].min()).nonzero()[:, 0]
        out = int(low[pos[s, low].argmax()])
        if out != m:
            k[:, s, :, out], v[:, s, :, out] = k_new[:, s], v_new[:, s]
            ud[s, out], pos[s, out] = ud[s, m].clone(), cur
    r = {"k": k[:, :, :, :m].double(), "v": v[:, :, :, :m].double(), "u": ud[:, :m], "pos": pos[:, :m]}
    if case.get("variant") == "vnorm":
        r["norms"] = v[:, :, :, :m].double().norm(dim=-1)
    if kind == "decode":
        r["o"] = torch.stack(o)
    return r
