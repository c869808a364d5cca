"""The work a decode engine has this library do, as cases whose time can be measured.

``listed()`` names them, ``draw()`` gives more of the same ranges, ``prepare()`` makes what
a program holds before the call, ``run()`` is one pass through the package's public entry
points, ``exact()`` the same outputs in 64 bits from plain torch.

Kinds of case:

* ``step``     one decode step of a stack of layers (``DecodeStack.step``): every schedule,
               page size, head shape, data type and metadata kind that is used in earnest.
               Queries follow an AR(1) process back and forth along a short trajectory, so
               that consecutive steps select overlapping pages, as decode steps do.
* ``prefill``  the end of a prompt: page metadata of every layer, then step 0.
* ``attend``   attention over given page lists, layer by layer (``LayerState.repair``).
* ``merge``    partial states of several shards merged (``prr_merge_states``).
* ``calibrate`` the host-side EMA calibration of one layer (``prr_calibrate``).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_30389_amd import _lib as L
from paper_2606_30389_amd import runtime as R

DEV = "cuda:0"
D = 128
TRAJECTORY = 12  # queries of a step case, walked back and forth

SCHEDULES = {
    "prr": L.PRR_SCHED_FUSED_PRR,
    "fused_serial": L.PRR_SCHED_FUSED_SERIAL,
    "serial": L.PRR_SCHED_SERIAL,
    "two_stream": L.PRR_SCHED_TWO_STREAM,
}
THETAS = {"default": (0.5, 0.5, 0.0), "calibrated": (0.8, 0.5, 0.25)}


def _step(name, **kw):
    c = dict(kind="step", schedule="prr", hq=32, hkv=2, dtype="bf16", page=16, tokens=131072, budget=4096,
             forced="none", meta="minmax", layers=40, paged=False, mode="exact", theta="default")
    c.update(kw)
    return dict(c, name=name)


def listed():
    return [
        # the smallest call: one layer of a small model at a short context
        _step("tiny_step", hq=4, hkv=1, dtype="f16", tokens=2048, budget=256, layers=1),
        # a 40-layer model with two KV heads at 32K tokens, first and last page always kept
        _step("glm32k_step", tokens=32768, budget=2048, forced="first_last"),
        # the benchmark's workload: the same model at 128K tokens
        _step("glm128k_step"),
        # eight KV heads, half precision, the cache behind a page table
        _step("llama64k_step", hkv=8, dtype="f16", tokens=65536, budget=2048, layers=32, paged=True),
        # 64-token blocks ranked by their mean key, initial and local blocks on top of the budget
        _step("infllm128k_step", page=64, forced="initial_local2", meta="mean"),
        # select, then attend: the step without speculation, at a ragged length
        _step("glm100k_serial", schedule="fused_serial", tokens=100003),
        # a context beyond the fused step's 8192 pages: the step kernel by kernel
        _step("llama256k_serial", schedule="serial", hkv=8, dtype="f16", tokens=262144, layers=8),
        # 128-token pages: speculation beside selection on two streams
        _step("llama128k_p128_two_stream", schedule="two_stream", hkv=8, dtype="f16", page=128, layers=8),
        # the end of a 128K prompt: every layer's page metadata, then step 0
        dict(_step("glm128k_prefill"), kind="prefill", schedule="prefill"),
        # block-sparse attention over given lists of 32-token pages
        dict(_step("llama128k_p32_attend", hkv=8, dtype="f16", page=32, layers=8), kind="attend", schedule="attend"),
        # states of 64 context shards of one layer's 32 heads
        dict(name="merge_64_shards", kind="merge", states=64, rows=32, d=128),
        # one layer's calibration on 64 prefill rows of 8192 blocks
        dict(name="glm128k_calibrate", kind="calibrate", rows=64, blocks=8192, k=256, growing=4),
    ]


# ------------------------------------------------------------------------------- draws

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["prr", "fused_serial", "serial", "two_stream", "prefill", "attend", "merge", "calibrate"],
                       [6, 2, 1, 2, 1, 1, 1, 1])[0]
    if kind == "merge":
        return dict(kind="merge", states=_log_int(rng, 2, 256), rows=rng.choice([1, 8, 28, 32, 64]),
                    d=rng.choice([64, 128, 128, 192]))
    if kind == "calibrate":
        blocks = _log_int(rng, 256, 8192)
        return dict(kind="calibrate", rows=_log_int(rng, 16, 64), blocks=blocks, k=_log_int(rng, 8, max(9, blocks // 16)),
                    growing=rng.randrange(0, 8))
    fused = kind in ("prr", "fused_serial")
    page = rng.choice([16, 16, 16, 64]) if fused or kind == "prefill" else rng.choice([16, 32, 64, 128, 256])
    # the fused schedules take 8192 pages, the others 16384
    tokens = _log_int(rng, 2048, 131072 if page == 16 and (fused or kind == "prefill") else 262144)
    pages = -(-tokens // page)
    hkv = rng.choice([1, 2, 4, 8])
    group = rng.choice([g for g in (1, 4, 7, 8, 16) if g * hkv <= 64])
    # budgets as they are used: 1/16 of a short context to 4K tokens of a long one
    budget = min(_log_int(rng, 512, 4096), max(4 * page, tokens // 8))
    # a state holds no more than the largest listed one
    per_layer = hkv * pages * page * D * 4
    layers = max(1, min(_log_int(rng, 4, 40), int(8.5e9 // per_layer)))
    return dict(kind=kind if kind in ("prefill", "attend") else "step", schedule=kind, hq=hkv * group, hkv=hkv,
                dtype=rng.choice(["bf16", "f16"]), page=page, tokens=tokens, budget=budget,
                forced=rng.choice(["none", "first_last", "initial_local2"]),
                meta="minmax" if page < 64 else rng.choice(["minmax", "mean"]), layers=layers,
                paged=rng.choice([False, True]), mode="keep" if kind == "prr" and rng.random() < 0.2 else "exact",
                theta=rng.choice(["default", "calibrated"]))


# ------------------------------------------------------------------------------- inputs

def _pages(c):
    return -(-c["tokens"] // c["page"])


def _k_select(c):
    return max(1, min(c["budget"] // c["page"], _pages(c)))


def _forced(c):
    n = _pages(c)
    return {"none": [], "first_last": sorted({0, n - 1}), "initial_local2": sorted({0, max(0, n - 2), n - 1})}[c["forced"]]


def _in_budget(c):
    return c["forced"] != "initial_local2"  # initial and local blocks come on top of the budget


def _chunk(c):
    """Pages per attending workgroup: 128 tokens of speculation, 64 (at 16-token pages) or
    128 where every page is attended after the selection."""
    if c["schedule"] == "fused_serial":
        return {16: 4, 64: 2}[c["page"]]
    return max(1, 128 // c["page"])


def _torch_dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float16


def _config(c):
    theta = THETAS[c["theta"]]
    # the cache of a paged program has room for more than one prompt
    max_pages = _pages(c) + (max(8, _pages(c) // 16) if c["paged"] else 0)
    return R.PathConfig(num_q_heads=c["hq"], num_kv_heads=c["hkv"], page_size=c["page"], num_tokens=c["tokens"],
                        k_select=_k_select(c), forced=_forced(c), forced_in_budget=_in_budget(c), dtype=c["dtype"],
                        meta_kind=c["meta"], alpha=theta[0], beta=theta[1], gamma=theta[2], chunk_pages=_chunk(c),
                        mode=L.PRR_KEEP_WASTED if c["mode"] == "keep" else L.PRR_EXACT_SELECTED, max_pages=max_pages)


def _cache(c, seed):
    """Keys and values of every layer [layers][hkv][slots][page][128], the page table, the
    query trajectory [TRAJECTORY][layers][hq][128] and random page lists: N(0, 1) values with
    1% of the pages' keys shifted along one direction, AR(1) queries."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, dt, page = _pages(c), _torch_dtype(c), c["page"]
    slots = _config(c).max_pages
    shape = (c["layers"], c["hkv"], slots, page, D)
    k = torch.randn(shape, generator=g, dtype=dt, device=DEV)
    v = torch.randn(shape, generator=g, dtype=dt, device=DEV)
    table = torch.randperm(slots, generator=g, device=DEV)[:n] if c["paged"] else torch.arange(n, device=DEV)
    u = torch.randn(c["layers"], c["hkv"], D, generator=g, device=DEV)
    u = 2.0 * u / u.norm(dim=-1, keepdim=True)
    hot = torch.randint(0, n, (c["layers"], c["hkv"], max(1, n // 100)), generator=g, device=DEV)
    for i in range(c["layers"]):
        for h in range(c["hkv"]):
            p = table[hot[i, h].unique()]
            k[i, h, p] = (k[i, h, p].float() + u[i, h]).to(dt)
    q = torch.empty(TRAJECTORY, c["layers"], c["hq"], D, dtype=dt, device=DEV)
    x = torch.randn(c["layers"], c["hq"], D, generator=g, device=DEV)
    for t in range(TRAJECTORY):
        q[t] = x.to(dt)
        x = 0.95 * x + math.sqrt(1 - 0.95 ** 2) * torch.randn(x.shape, generator=g, device=DEV)
    kk = _k_select(c)
    r = torch.rand(c["layers"], c["hkv"], n, generator=g, device=DEV)
    lists = r.topk(kk, dim=-1).indices.sort(dim=-1).values.to(torch.int32)
    return k, v, table.to(torch.int32), q, lists


def _states(c, seed):
    """The inputs in an engine's layer states, whose results lie stacked in one tensor each."""
    k, v, table, q, lists = _cache(c, seed)
    cfg = _config(c)
    layers = [R.LayerState(cfg, DEV, k=k[i], v=v[i], page_table=table if c["paged"] else None)
              for i in range(c["layers"])]
    out = {}
    for name in ("out_o32", "out_o", "out_m", "out_l", "scores", "level", "trend", "init_bits", "meta", "sel", "missed",
                 "wasted"):
        out[name] = torch.stack([getattr(st, name) for st in layers])
        for i, st in enumerate(layers):
            setattr(st, name, out[name][i])
    for j in range(2):
        out["pred%d" % j] = torch.stack([st.pred[j] for st in layers])
        for i, st in enumerate(layers):
            st.pred[j] = out["pred%d" % j][i]
    return layers, out, q, lists


def _scores_trajectory(c, seed):
    r = np.random.default_rng(seed)
    x = r.standard_normal(c["blocks"])
    rows = []
    for _ in range(c["rows"]):
        rows.append(45.0 + 3.0 * x)
        x = 0.95 * x + math.sqrt(1 - 0.95 ** 2) * r.standard_normal(c["blocks"])
    form = np.zeros(c["blocks"], dtype=np.int32)
    for i in range(c["growing"]):  # the prompt's last blocks form along the trajectory
        form[c["blocks"] - 1 - i] = max(0, c["rows"] - 1 - i * c["rows"] // 8)
    return np.stack(rows).astype(np.float32), form


def _merge_inputs(c, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    o = torch.randn(c["states"], c["rows"], c["d"], generator=g, device=DEV)
    m = 3.0 + torch.randn(c["states"], c["rows"], generator=g, device=DEV)
    l = 1.0 + 100.0 * torch.rand(c["states"], c["rows"], generator=g, device=DEV)
    # a shard without a selected page hands in the empty state
    empty = torch.rand(c["states"], c["rows"], generator=g, device=DEV) < 0.1
    empty[0] = False
    return torch.where(empty[..., None], 0.0, o), torch.where(empty, -math.inf, m), torch.where(empty, 0.0, l)


def prepare(case, seed):
    c = case
    if c["kind"] == "merge":
        o, m, l = _merge_inputs(c, seed)
        return dict(kind="merge", case=c, o=o, m=m, l=l, out=(torch.empty_like(o[0]), torch.empty_like(m[0]), torch.empty_like(l[0])))
    if c["kind"] == "calibrate":
        scores, form = _scores_trajectory(c, seed)
        # 16 threads: the share of the host that one GPU's process has
        return dict(kind="calibrate", case=c, scores=scores, form=form, grid=np.asarray(R.THETA_GRID, dtype=np.float32), threads=16)
    layers, out, q, lists = _states(c, seed)
    stream = torch.cuda.current_stream()
    s = dict(kind=c["kind"], case=c, layers=layers, out=out, q=q, t=0)
    if c["kind"] == "attend":
        for i, st in enumerate(layers):
            st.sel[:, :lists.shape[-1]] = lists[i]
            st.sel_count.fill_(lists.shape[-1])
        return s
    stack = R.DecodeStack(layers, [q[0, i] for i in range(c["layers"])], DEV)
    stack.params.late_spec = 1 if c["schedule"] == "prr" else 0
    s["stack"] = stack
    if c["kind"] == "prefill":
        return s
    # the prompt is in: metadata built, EMA state and first prediction from its last query
    for st in layers:
        st.build_meta()
    fused = c["schedule"] in ("prr", "fused_serial")
    stack.step(L.PRR_SCHED_FUSED_PREFILL if fused else L.PRR_SCHED_PREFILL, stream)
    # the steps' layer descriptors, one set per query of the trajectory
    s["io"] = [(L.prr_layer_io * c["layers"])(*[st.io(q[t, i]) for i, st in enumerate(layers)]) for t in range(TRAJECTORY)]
    if c["schedule"] == "two_stream":
        s["spec_stream"] = torch.cuda.Stream()
    return s


def run(state):
    s = state
    if s["kind"] == "merge":
        L.prr_merge_states(s["case"]["states"], s["case"]["rows"], s["case"]["d"], s["o"], s["m"], s["l"], *s["out"])
        return s["out"]
    if s["kind"] == "calibrate":
        theta, objective = L.prr_calibrate(s["scores"], s["case"]["k"], s["grid"], n_threads=s["threads"], form_row=s["form"])
        return theta, objective
    out, stream = s["out"], torch.cuda.current_stream()
    if s["kind"] == "attend":
        for i, st in enumerate(s["layers"]):
            st.repair(s["q"][0, i], stream=stream, serial=True)
        return {n: out[n] for n in ("out_o32", "out_o", "out_m", "out_l")}
    stack = s["stack"]
    if s["kind"] == "prefill":
        out["init_bits"].zero_()  # a new prompt
        for st in s["layers"]:
            st.build_meta(stream=stream)
        stack.step(L.PRR_SCHED_FUSED_PREFILL, stream)
        return {n: out[n] for n in ("meta", "scores", "level", "trend", "sel", "pred%d" % s["layers"][0].cur)}
    s["t"] += 1
    t = s["t"] % (2 * TRAJECTORY - 2)
    stack.io = s["io"][t if t < TRAJECTORY else 2 * TRAJECTORY - 2 - t]
    schedule = s["case"]["schedule"]
    stack.step(SCHEDULES[schedule], stream, s.get("spec_stream"))
    names = ["out_o32", "out_o", "out_m", "out_l", "scores", "sel"]
    if schedule in ("prr", "two_stream"):
        names += ["level", "trend", "missed", "wasted", "pred%d" % s["layers"][0].cur]
    return {n: out[n] for n in names}


# ------------------------------------------------------------------------------- work

def work(case):
    c = case
    if c["kind"] == "merge":
        n = c["states"] * c["rows"]
        return {"bytes": (n + c["rows"]) * (c["d"] + 2) * 4, "flops": 2 * n * c["d"]}
    if c["kind"] == "calibrate":
        # per grid point, row and block: prediction (2), trend and level (4 each); the ranking
        # of a row counts as one operation per block
        n = c["rows"] * c["blocks"]
        return {"bytes": 4 * n, "flops": 11 * n * len(R.THETA_GRID)}
    n, hkv, hq, kk = _pages(c), c["hkv"], c["hq"], _k_select(c)
    picked = kk + (0 if _in_budget(c) else len(_forced(c)))
    meta, scores, ema = hkv * n * 512, hkv * n * 4, hkv * n * 16
    kv = 2 * hkv * picked * c["page"] * D * 2
    qo = hq * D * (2 + 4 + 2) + hq * 8
    attend_flops = 4 * hq * picked * c["page"] * D
    score_flops = 4 * hkv * n * D
    if c["kind"] == "attend":
        b, f = kv + qo, attend_flops
    elif c["kind"] == "prefill":
        b, f = hkv * c["tokens"] * D * 2 + 2 * meta + scores + ema // 2, hkv * c["tokens"] * D * 2 + score_flops
    elif c["schedule"] in ("prr", "two_stream"):
        b, f = meta + scores + ema + kv + qo, score_flops + attend_flops
    else:
        b, f = meta + scores + kv + qo, score_flops + attend_flops
    return {"bytes": c["layers"] * b, "flops": c["layers"] * f}


def tolerance(case):
    c = case
    if c["kind"] == "merge":
        return {"rel": 2e-6, "max": 1e-5}
    if c["kind"] == "calibrate":
        # sums of doubles in another order
        return {"rel": 1e-12, "max": 1e-11}
    # 32-bit sums; out_o is the 32-bit output rounded to 16 bits, where a last bit of the
    # sum moves one value in about a thousand by a unit of its last place (2^-8)
    return {"rel": 2e-4, "max": 8e-3}


# ------------------------------------------------------------------------------- 64 bits

def _page_bounds(c, k, table):
    """Logical pages' (min, max) or mean of the valid tokens, one KV head, in 64 bits."""
    x = k[table.long()].double()
    tail = c["tokens"] - (x.shape[0] - 1) * c["page"]
    if c["meta"] == "mean":
        mean = x.mean(dim=1)
        mean[-1] = x[-1, :tail].mean(dim=0)
        return mean, mean
    lo, hi = x.amin(dim=1), x.amax(dim=1)
    lo[-1], hi[-1] = x[-1, :tail].amin(dim=0), x[-1, :tail].amax(dim=0)
    return lo, hi


def _top(scores, c):
    forced = _forced(c)
    kk = max(0, _k_select(c) - len(forced)) if _in_budget(c) else _k_select(c)
    x = scores.clone()
    x[forced] = -math.inf
    kk = min(kk, x.numel() - len(forced))
    return torch.cat([torch.tensor(forced, device=DEV, dtype=torch.int64), x.topk(kk).indices]).sort().values


def _attention(c, q, k, v, table, pages):
    """(o, m, l) of the G query heads of one KV head over the tokens of `pages`."""
    x, y = k[table[pages].long()].double().reshape(-1, D), v[table[pages].long()].double().reshape(-1, D)
    token = (pages[:, None] * c["page"] + torch.arange(c["page"], device=DEV)).reshape(-1)
    s = (q.double() @ x.T) / math.sqrt(D)
    s = s.masked_fill(token >= c["tokens"], -math.inf)
    m = s.amax(dim=-1)
    p = (s - m[:, None]).exp()
    l = p.sum(dim=-1)
    return (p @ y) / l[:, None], m, l


def _exact_merge(c, seed):
    o, m, l = (x.double() for x in _merge_inputs(c, seed))
    top = m.amax(dim=0)
    w = l * (m - top).exp()
    total = w.sum(dim=0)
    return (w[..., None] * o).sum(dim=0) / total[:, None], top, total


def _exact_calibrate(c, seed):
    scores, form = _scores_trajectory(c, seed)
    scores = scores.astype(np.float64)

    def top(x, k, exists):
        key = np.where(exists, x, -np.inf).astype(np.float32)
        picked = np.argsort(-key, kind="stable")[:min(k, int(exists.sum()))]
        mask = np.zeros(len(x), dtype=bool)
        mask[picked] = True
        return mask

    chosen = [top(scores[t], c["k"], form <= t) for t in range(c["rows"])]
    objective = []
    for a, b, g in np.asarray(R.THETA_GRID, dtype=np.float32).astype(np.float64):
        level, trend, has, rates = np.zeros(c["blocks"]), np.zeros(c["blocks"]), np.zeros(c["blocks"], dtype=bool), []
        for t in range(c["rows"]):
            x = scores[t]
            if t:
                hit = chosen[t] & top(level + g * trend, c["k"], has)
                rates.append(x[hit].sum() / x[chosen[t]].sum())
                trend = np.where(has, b * (x - level) + (1 - b) * trend, trend)
                level = np.where(has, a * x + (1 - a) * level, level)
            new = ~has & (form <= t)
            level, trend, has = np.where(new, x, level), np.where(new, 0.0, trend), has | new
        objective.append(np.mean(rates))
    return None, np.asarray(objective)


def exact(case, seed):
    c = case
    if c["kind"] == "merge":
        return _exact_merge(c, seed)
    if c["kind"] == "calibrate":
        return _exact_calibrate(c, seed)
    k, v, table, q, lists = _cache(c, seed)
    n, slots, G = _pages(c), k.shape[2], c["hq"] // c["hkv"]
    theta = THETAS[c["theta"]]
    f64 = dict(dtype=torch.float64, device=DEV)
    o, m, l = torch.zeros(c["layers"], c["hq"], D, **f64), torch.zeros(c["layers"], c["hq"], **f64), torch.zeros(c["layers"], c["hq"], **f64)
    scores, level, trend = (torch.zeros(c["layers"], c["hkv"], slots, **f64) for _ in range(3))
    meta = torch.zeros(c["layers"], c["hkv"], slots, *((D,) if c["meta"] == "mean" else (2, D)), **f64) if c["kind"] == "prefill" else None
    for i in range(c["layers"]):
        for h in range(c["hkv"]):
            rows = slice(h * G, (h + 1) * G)
            if c["kind"] == "attend":
                o[i, rows], m[i, rows], l[i, rows] = _attention(c, q[0, i, rows], k[i, h], v[i, h], table, lists[i, h].long())
                continue
            lo, hi = _page_bounds(c, k[i, h], table)

            def score(t):
                qbar = q[t, i, rows].double().mean(dim=0)
                return lo @ qbar if c["meta"] == "mean" else torch.maximum(qbar * lo, qbar * hi).sum(dim=-1)

            s0 = score(0)
            if c["kind"] == "prefill":
                scores[i, h, :n] = level[i, h, :n] = s0
                meta[i, h, :n] = lo if c["meta"] == "mean" else torch.stack([lo, hi], dim=1)
                continue
            s1 = score(1)
            scores[i, h, :n] = s1
            level[i, h, :n] = theta[0] * s1 + (1 - theta[0]) * s0
            trend[i, h, :n] = theta[1] * (s1 - s0)
            pages = _top(s1, c)
            if c["mode"] == "keep":
                pages = torch.cat([pages, _top(s0, c)]).unique()
            o[i, rows], m[i, rows], l[i, rows] = _attention(c, q[1, i, rows], k[i, h], v[i, h], table, pages)
    if c["kind"] == "prefill":
        return {"meta": meta, "scores": scores, "level": level, "trend": trend}
    r = {"out_o32": o, "out_o": o, "out_m": m, "out_l": l}
    if c["kind"] == "step":
        r["scores"] = scores
        if c["schedule"] in ("prr", "two_stream"):
            r.update(level=level, trend=trend)
    return r
