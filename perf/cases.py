"""Performance cases of the episode-counting engine: the work its users have it do, through epi.py.

listed() are the cases, draw() gives more of the same ranges, prepare() makes what a program holds before
the call (inputs from the seed, a context, loaded streams, submitted candidates, a trained model), run() is
one pass, work() the bytes and operations a pass cannot do without, exact() its outputs in 64 bits.

The kinds of work:
  count    candidate sets on loaded streams counted again (plain, batched, allocation-free), counts read back;
  query    a new recording on the device: load and index it, submit candidates, count, read;
  append   a recording followed live: load its history, count, then chunks appended and counted incrementally;
  track    a few long episodes over a long stream, counted per event;
  mine     level-wise discovery on a loaded stream, the patterns of the last two levels asked for read back;
  model    the cost model: an epoch of training from given weights, then predictions for other samples.

Streams are spike trains: Poisson types of one rate, Zipf rates (a few busy types, many quiet ones) or bursty
ones (rates redrawn every second), with planted cascades; int32 microseconds or int64 nanoseconds.
"""
import math

import numpy as np
import torch

from paper_0905_2203_amd import epi

MENU_MS = ((0, 5), (5, 10), (10, 20))  # intervals of planted cascades and of level-wise discovery
LOW_MS, WIDTH_MS = (0, 5, 10, 20), (5, 10, 20)  # random candidates: (l, l + w]
MODES = {"plain": epi.EPI_MODE_PLAIN, "batched": epi.EPI_MODE_BATCHED}
SCHEDS = {"rr": epi.EPI_SCHED_RR, "learned": epi.EPI_SCHED_LEARNED, "heuristic": epi.EPI_SCHED_HEURISTIC}
MOST_VISITS = 3.2e10  # candidate-type events of the largest listed case


def listed():
    return [
        # every ordered pair of a short recording: the smallest interactive question, bound by launches
        dict(name="pairs_short", kind="count", proc="poisson", sets=1, n=10500, K=32, rate=10.0, ts="i32", m=992, nmin=2,
             nmax=2, mode="plain", sched="rr", repeats=False),
        # many recordings of very different lengths in one batched call, bursty and sparse (int64 ns)
        dict(name="recordings", kind="count", proc="bursty", sets=8, n=2200000, K=60, rate=15.0, ts="i64", m=41000, nmin=2,
             nmax=8, mode="batched", sched="heuristic", repeats=False),
        # a few busy types among many quiet ones, candidates ordered by the learned cost
        dict(name="zipf_learned", kind="count", proc="zipf", sets=1, n=2500000, K=128, rate=21.7, ts="i64", m=12500, nmin=3,
             nmax=8, mode="batched", sched="learned", repeats=False),
        # a mid-sized one-off count in microseconds, repeated types allowed
        dict(name="mid_plain", kind="count", proc="poisson", sets=1, n=1500001, K=101, rate=37.0, ts="i32", m=5003, nmin=1,
             nmax=6, mode="plain", sched="rr", repeats=True),
        # the large workload: 256 types at 50 Hz, tens of thousands of candidates of every size
        dict(name="large_batched", kind="count", proc="poisson", sets=1, n=20000000, K=256, rate=50.8, ts="i64", m=80000,
             nmin=2, nmax=8, mode="batched", sched="rr", repeats=False),
        # a new long recording queried once: ingest, index, a few candidates
        dict(name="query_new", kind="query", n=9000000, K=128, proc="zipf", rate=21.7, ts="i64", m=256, nmin=2, nmax=5),
        # a live recording: history, then a chunk every few seconds
        dict(name="append_live", kind="append", n=1200000, K=64, proc="poisson", rate=40.0, ts="i64", m=2000, nmin=2, nmax=6,
             chunks=6, chunk=20000),
        # a few long cascades in an hour of recording
        dict(name="track_long", kind="track", n=9400000, K=64, proc="poisson", rate=40.0, ts="i64", m=16, nmin=8, nmax=8,
             order=False),
        # level-wise discovery on five minutes of 64 channels, every chance triple kept (threshold 100)
        dict(name="mine_dense", kind="mine", n=416000, K=64, proc="poisson", rate=20.0, ts="i32", threshold=100, max_size=6),
        # discovery above chance on a minute of 40 channels
        dict(name="mine_short", kind="mine", n=50000, K=40, proc="poisson", rate=20.0, ts="i32", threshold=60, max_size=5),
        # an epoch of the cost model on the work log of a few thousand episodes
        dict(name="model_epoch", kind="model", m=8192, batch=512, predict=50000),
    ]


def _between(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def _one(rng):
    kind = rng.choice(("count", "count", "count", "query", "append", "track", "mine", "model"))
    if kind == "model":
        return dict(kind=kind, m=_between(rng, 1000, 8192), batch=rng.choice((256, 512, 512, 700)),
                    predict=_between(rng, 500, 50000))
    c = dict(kind=kind, proc=rng.choice(("poisson", "zipf", "bursty")), K=_between(rng, 24, 256),
             rate=round(rng.uniform(8, 55), 1), ts=rng.choice(("i32", "i64")))
    if kind == "count":
        lo = rng.randint(1, 4)
        c.update(sets=rng.choice((1, 1, 2, 5)), n=_between(rng, 10000, 20000000), m=_between(rng, 64, 80000), nmin=lo,
                 nmax=rng.randint(lo + 1, 8), mode=rng.choice(("plain", "batched", "batched", "noalloc")),
                 sched=rng.choice(("rr", "heuristic", "learned")), repeats=rng.random() < 0.2)
    elif kind == "query":
        c.update(n=_between(rng, 20000, 9000000), m=_between(rng, 16, 2000), nmin=2, nmax=rng.randint(3, 6))
    elif kind == "append":
        c.update(n=_between(rng, 50000, 1200000), m=_between(rng, 100, 2000), nmin=2, nmax=rng.randint(3, 7),
                 chunks=rng.randint(2, 6), chunk=_between(rng, 1000, 20000))
    elif kind == "track":
        lo = rng.randint(2, 8)
        c.update(n=_between(rng, 100000, 9400000), m=rng.randint(4, 24), nmin=lo, nmax=lo, order=rng.random() < 0.3)
    else:
        c.update(proc="poisson", K=rng.randint(24, 64), rate=20.0)
        dur = rng.uniform(40, 260)
        c.update(n=int(c["K"] * 20.0 * dur), threshold=int(dur * rng.uniform(0.4, 1.5)), max_size=rng.randint(4, 6))
    if c["ts"] == "i32":  # microseconds: at most 2000 s
        c["n"] = int(min(c["n"], 2000 * c["K"] * c["rate"]))
    return c


def draw(rng):
    while True:
        c = _one(rng)
        if c["kind"] != "count" or _visits(c) <= MOST_VISITS and _visits(c, busy=True) <= MOST_VISITS / 2:
            return c


def _visits(c, busy=False):
    """Events of the candidates' types, summed over the candidates (busy: skewed rates weigh more)."""
    v = c["m"] * 0.5 * (c["nmin"] + c["nmax"]) * c["n"] / c["K"] / c.get("sets", 1)
    return v * (4 if busy and c["proc"] == "zipf" else 1)


# ---- inputs -----------------------------------------------------------------
def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _stream(c, seed, n):
    """types int32[n], times (int32 us or int64 ns) on the GPU, planted cascades as (types, intervals in ms)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    K, unit = c["K"], 1000 if c["ts"] == "i32" else 1000000
    dur = max(1.0, n / (K * c["rate"]))  # seconds
    host = np.random.Generator(np.random.PCG64(int(seed)))
    pool, planted, parts = host.permutation(K), [], []
    for size in host.integers(3, 7, size=max(1, min(8, K // 16))):
        ty, pool = pool[:size], pool[size:]
        planted.append((ty, [MENU_MS[i] for i in host.integers(0, 3, size=size - 1)]))
    left = n
    for ty, gaps in planted:
        k = min(int(host.uniform(2, 8) * dur), left // 8 // len(ty))
        t = _rand(g, k) * (dur * 1000 * unit)
        t = t.floor_().long()
        for j in range(len(ty)):
            if j:
                lo, hi = gaps[j - 1]
                t = t + torch.randint(lo * unit + 1, hi * unit + 1, (k,), generator=g, device="cuda")
            parts.append((torch.full((k,), int(ty[j]), dtype=torch.int32, device="cuda"), t))
        left -= k * len(ty)
    if c["proc"] == "poisson":
        ty = torch.randint(0, K, (left,), generator=g, device="cuda")
        t = _rand(g, left) * dur
    elif c["proc"] == "zipf":
        p = torch.arange(1, K + 1, dtype=torch.float64, device="cuda") ** -1.2
        ty = torch.searchsorted(torch.cumsum(p / p.sum(), 0), _rand(g, left)).clamp_(max=K - 1)
        t = _rand(g, left) * dur
    else:  # each type's rate redrawn every second, Gamma(2)
        win = max(1, int(dur))
        p = torch.cumsum(-(_rand(g, win * K) * _rand(g, win * K)).clamp_(min=1e-300).log_(), 0)
        cell = torch.searchsorted(p, _rand(g, left) * p[-1]).clamp_(max=win * K - 1)
        ty, t = cell % K, ((cell // K) + _rand(g, left)) * (dur / win)
    parts.append((ty.int(), (t * (1000.0 * unit)).floor_().long()))
    ty, t = torch.cat([a for a, _ in parts]), torch.cat([b for _, b in parts])
    t, order = torch.sort(t)
    ty = ty[order].contiguous()
    return ty, t.int() if c["ts"] == "i32" else t, planted


def _candidates(c, seed, m, planted):
    """m random episodes over the interval menu, the planted cascades' prefixes first."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 7919)
    host = np.random.Generator(np.random.PCG64([int(seed), 1]))
    unit = 1000 if c["ts"] == "i32" else 1000000
    if c.get("repeats"):
        ty = torch.randint(0, c["K"], (m, 8), generator=g, device="cuda")
    else:
        ty = torch.rand(m, c["K"], generator=g, device="cuda").topk(8, dim=1).indices
    N = host.integers(c["nmin"], c["nmax"] + 1, size=m)
    lo = np.asarray(LOW_MS)[host.integers(0, len(LOW_MS), size=(m, 7))]
    hi = lo + np.asarray(WIDTH_MS)[host.integers(0, len(WIDTH_MS), size=(m, 7))]
    ty = ty.cpu().numpy().astype(np.int32)
    i = 0
    for types, gaps in planted:
        for size in range(max(2, c["nmin"]), min(len(types), c["nmax"]) + 1):
            if i < m // 2:
                N[i], ty[i, :size] = size, types[:size]
                lo[i, : size - 1], hi[i, : size - 1] = [a for a, _ in gaps[: size - 1]], [b for _, b in gaps[: size - 1]]
                i += 1
    ty = np.where(np.arange(8)[None, :] < N[:, None], ty, -1)
    live = np.arange(7)[None, :] < N[:, None] - 1
    return dict(N=N.astype(np.uint8), types=np.ascontiguousarray(ty, np.int32),
                lo=np.where(live, lo * unit, 0).astype(np.int64), hi=np.where(live, hi * unit, 0).astype(np.int64))


def _shares(total, parts, seed):
    """`total` in `parts` unequal shares (log-uniform over a factor of twenty), the same for every seed."""
    w = np.exp(np.random.Generator(np.random.PCG64([parts, seed])).uniform(0, math.log(20), size=parts))
    return [max(64, int(total * x / w.sum())) for x in w]


def _inputs(c, seed):
    """The streams and candidate sets of a case."""
    k = c.get("sets", 1)
    ns = [c["n"]] if k == 1 else _shares(c["n"], k, 1)
    ms = [c["m"]] if k == 1 else _shares(c["m"], k, 2)
    out = []
    for i in range(k):
        ty, t, planted = _stream(c, seed * 64 + i, ns[i])
        out.append((ty, t, _candidates(c, seed * 64 + i, ms[i], planted)))
    return out


def _samples(c, seed):
    """Standardised features, targets and He-uniform weights of the cost model."""
    r = np.random.Generator(np.random.PCG64([int(seed), 3]))
    X = r.standard_normal((c["m"] + c["predict"], 24)).astype(np.float32)
    t = (0.5 * X[:, 23] * X[:, 0] + np.sin(X[:, 3]) - 0.3 * X[:, 7] + 0.1 * r.standard_normal(X.shape[0])).astype(np.float32)
    p = [r.uniform(-1, 1, (24, 64)) * math.sqrt(6 / 24), np.zeros(64), r.uniform(-1, 1, (64, 64)) * math.sqrt(6 / 64),
         np.zeros(64), r.uniform(-1, 1, 64) * math.sqrt(6 / 64), np.zeros(1)]
    p = np.concatenate([x.ravel() for x in p]).astype(np.float32)
    return X[: c["m"]], t[: c["m"]], p, np.ascontiguousarray(X[c["m"]:])


def _patterns(c, sizes, found):
    """Outputs of a discovery: (candidates, frequent) of every level asked for, and the patterns found of the last
    two in tables that hold any number of them (unused rows 0)."""
    out = [np.array(sizes + [(0, 0)] * (c["max_size"] - len(sizes)), np.int64)]
    for level in (c["max_size"] - 1, c["max_size"]):
        types, lo, hi, counts = found.get(level, (np.zeros((0, 8)), np.zeros((0, 7)), np.zeros((0, 7)), np.zeros(0)))
        f, rows = len(counts), c["K"] ** 3 * (9 if level <= 3 else 2)
        if f > rows:
            raise ValueError("more patterns than the table holds")
        t = dict(types=np.zeros((rows, 8), np.int32), lo=np.zeros((rows, 7), np.int64), hi=np.zeros((rows, 7), np.int64),
                 counts=np.zeros(rows, np.int32))
        t["types"][:f], t["lo"][:f], t["hi"][:f], t["counts"][:f] = types, lo, hi, counts
        out.append(t)
    return out


# ---- cases -------------------------------------------------------------------
def prepare(case, seed):
    c, s = case, dict(case=case, ctx=epi.Context(0))
    ctx = s["ctx"]
    if c["kind"] == "model":
        s["X"], s["t"], s["p"], s["Xp"] = _samples(c, seed)
        ctx.epi_mlp_init(24, 1)
        return s
    if c["kind"] == "mine":
        ty, t, _ = _stream(c, seed, c["n"])
        torch.cuda.synchronize()
        s["sid"] = ctx.epi_load_stream_device(ty, t, c["K"])
        unit = 1000 if c["ts"] == "i32" else 1000000
        s["menu"] = [(a * unit, b * unit) for a, b in MENU_MS]
        return s
    if c.get("repeats"):
        ctx.epi_set_option(epi.EPI_OPT_ALLOW_REPEATS, 1)
    if c.get("order"):
        ctx.epi_set_option(epi.EPI_OPT_STREAM_ORDER, 1)
    if c["kind"] in ("query", "append"):
        extra = c.get("chunks", 0) * c.get("chunk", 0)
        ty, t, planted = _stream(c, seed, c["n"] + extra)
        s["cands"] = _candidates(c, seed, c["m"], planted)
        if c["kind"] == "append":
            ty, t = ty.cpu().numpy(), t.cpu().numpy()
        s["types"], s["times"] = ty, t
        torch.cuda.synchronize()
        return s
    s["sets"], s["m"] = [], []
    for ty, t, cands in _inputs(c, seed):
        torch.cuda.synchronize()
        sid = ctx.epi_load_stream_device(ty, t, c["K"])
        s["sets"].append(ctx.epi_submit_candidates(sid, cands))
        s["m"].append(cands["N"].size)
    if c.get("sched") == "learned" and c["mode"] == "batched":  # a model trained on the log of a small set
        small = _candidates(c, seed + 1, min(512, c["m"]), [])
        tid = ctx.epi_submit_candidates(sid, small)
        ctx.epi_set_option(epi.EPI_OPT_WORKLOG, 1)
        ctx.epi_count([tid])
        ctx.epi_costmodel_train([tid], 8, 1)
        ctx.epi_set_option(epi.EPI_OPT_WORKLOG, 0)
        ctx.epi_release_set(tid)
    return s


def run(s):
    c, ctx = s["case"], s["ctx"]
    if c["kind"] == "count":
        if c["mode"] == "noalloc":
            for i in s["sets"]:
                ctx.epi_count_noalloc(i)
        else:
            ctx.epi_count(s["sets"], MODES[c["mode"]], SCHEDS[c["sched"]])
        return [ctx.epi_read_counts(i, m) for i, m in zip(s["sets"], s["m"])]
    if c["kind"] == "track":
        ctx.epi_count(s["sets"], epi.EPI_MODE_TRACKING)
        return [ctx.epi_read_counts(s["sets"][0], c["m"])]
    if c["kind"] == "query":
        sid = ctx.epi_load_stream_device(s["types"], s["times"], c["K"])
        cid = ctx.epi_submit_candidates(sid, s["cands"])
        ctx.epi_count([cid])
        counts = ctx.epi_read_counts(cid, c["m"])
        ctx.epi_release_set(cid)
        ctx.epi_release_stream(sid)
        return [counts]
    if c["kind"] == "append":
        n, out = c["n"], []
        sid = ctx.epi_load_stream(s["types"][:n], s["times"][:n], c["K"])
        cid = ctx.epi_submit_candidates(sid, s["cands"])
        ctx.epi_count([cid])
        out.append(ctx.epi_read_counts(cid, c["m"]))
        for k in range(c["chunks"]):
            a, b = n + k * c["chunk"], n + (k + 1) * c["chunk"]
            ctx.epi_append_stream(sid, s["types"][a:b], s["times"][a:b])
            ctx.epi_count([cid], epi.EPI_MODE_INCREMENTAL)
            out.append(ctx.epi_read_counts(cid, c["m"]))
        ctx.epi_release_set(cid)
        ctx.epi_release_stream(sid)
        return out
    if c["kind"] == "mine":
        mid = ctx.epi_mine(s["sid"], s["menu"], c["max_size"], c["threshold"])
        levels, found = range(1, ctx.epi_mine_levels(mid) + 1), {}
        sizes = [ctx.epi_mine_level_info(mid, level)[:2] for level in levels]
        for level in levels[c["max_size"] - 2:]:
            e, counts = ctx.epi_mine_read(mid, level, frequent_only=True)
            found[level] = (e["types"], e["lo"], e["hi"], counts)
        ctx.epi_mine_release(mid)
        return _patterns(c, sizes, found)
    ctx.epi_mlp_set_params(s["p"])
    losses = ctx.epi_mlp_train(s["X"], s["t"], 1, c["batch"], 3e-3)
    return [losses, ctx.epi_mlp_get_params(), ctx.epi_mlp_forward(s["Xp"])]


def work(case):
    c = case
    if c["kind"] == "model":
        per = 2 * (24 * 64 + 64 * 64 + 64)
        params = 24 * 64 + 64 + 64 * 64 + 64 + 64 + 1
        steps = -(-c["m"] // c["batch"])
        return dict(bytes=4 * (25 * (c["m"] + c["predict"]) + 6 * params * steps), flops=3 * per * c["m"] + per * c["predict"])
    tb = 4 if c["ts"] == "i32" else 8
    if c["kind"] == "mine":  # the stream once per level; a candidate takes its count and the test of its end events
        return dict(bytes=c["max_size"] * c["n"] * (tb + 4.0), flops=3.0 * c["max_size"] * c["n"] * c["K"])
    once = 146.0 * c["m"] + c["n"] * tb  # candidates, their counts, and the events of the index
    v = _visits(c)
    if c["kind"] == "query":  # the events as they come, and the index written
        once += c["n"] * (tb + 8.0)
    if c["kind"] == "append":
        v = v * (1 + c["chunks"] * c["chunk"] / c["n"])
        once += (c["n"] + c["chunks"] * c["chunk"]) * (tb + 8.0) + 4.0 * c["m"] * c["chunks"]
    return dict(bytes=once, flops=v)


# ---- 64-bit values -------------------------------------------------------------
def _extend(chain, times, lo, hi):
    """End events and latest starts of a chain extended by one node with the given event times."""
    ends, starts = chain
    i = np.searchsorted(ends, times - lo, side="left") - 1  # latest end before t - lo
    ok = i >= 0
    ok[ok] = times[ok] - ends[i[ok]] <= hi
    return times[ok], starts[i[ok]]


def _greedy(chain):
    """Most non-overlapped occurrences: each next one starts after the last one's end."""
    ends, starts = chain
    if not ends.size:
        return 0
    nxt = np.searchsorted(starts, ends, side="right").tolist()
    i, k, n = 0, 0, ends.size
    while i < n:
        i, k = nxt[i], k + 1
    return k


def _lists(types, times, K):
    order = np.argsort(types, kind="stable")
    cut = np.searchsorted(types[order], np.arange(K + 1))
    by = times.astype(np.int64)[order]
    return [by[cut[k]:cut[k + 1]] for k in range(K)]


def _counts(by, cands):
    out = np.zeros(cands["N"].size, np.int32)
    for i, n in enumerate(cands["N"]):
        t = by[cands["types"][i, 0]]
        chain = (t, t)
        for j in range(1, n):
            chain = _extend(chain, by[cands["types"][i, j]], cands["lo"][i, j - 1], cands["hi"][i, j - 1])
        out[i] = _greedy(chain)
    return out


def _levels(by, menu, max_size, threshold, most=60000):
    """Level-wise discovery; None when a level has more than `most` candidates."""
    K, out, prev = len(by), [], []
    for size in range(1, max_size + 1):
        if size == 1:
            cand = [((k,), (), (by[k], by[k]), -1) for k in range(K)]
        elif size == 2:
            cand = [(a + b, (v,), None, i) for i, (a, _, _, _) in enumerate(prev) for b, _, _, _ in prev if a != b
                    for v in range(len(menu))]
        else:
            tails = {}
            for ty, iv, _, _ in prev:
                tails.setdefault((ty[:-1], iv[:-1]), []).append((ty[-1], iv[-1]))
            cand = [(ty + (t,), iv + (v,), None, i) for i, (ty, iv, _, _) in enumerate(prev)
                    for t, v in tails.get((ty[1:], iv[1:]), ()) if t != ty[0]]
        if size > 1 and not cand:
            break
        if len(cand) > most:
            return None
        keep = []
        for ty, iv, chain, i in cand:
            if chain is None:
                chain = _extend(prev[i][2], by[ty[-1]], *menu[iv[-1]])
            k = _greedy(chain)
            if k > threshold:
                keep.append(((ty, iv, chain, i), k))
        f = len(keep)
        types, lo, hi = np.full((f, 8), -1, np.int32), np.zeros((f, 7), np.int64), np.zeros((f, 7), np.int64)
        for r, ((ty, iv, _, _), _) in enumerate(keep):
            types[r, :size] = ty
            lo[r, : size - 1], hi[r, : size - 1] = [menu[v][0] for v in iv], [menu[v][1] for v in iv]
        out.append((len(cand), f, types, lo, hi, np.array([k for _, k in keep], np.int32)))
        prev = [x for x, _ in keep]
        if not prev or size == 1 and f < 2:
            break
    return out


def _epoch(X, t, p, batch, lr):
    """One epoch of mini-batch Adam on the mean squared error, in 64 bits."""
    X, t, p = X.astype(np.float64), t.astype(np.float64), p.astype(np.float64)
    m, v, total, lr = np.zeros_like(p), np.zeros_like(p), 0.0, float(np.float32(lr))
    for k, b in enumerate(range(0, len(t), batch)):
        x, y = X[b:b + batch], t[b:b + batch]
        W1, b1, W2, b2, w3, b3 = _split(p)
        z1 = x @ W1 + b1
        h1 = np.maximum(z1, 0)
        z2 = h1 @ W2 + b2
        h2 = np.maximum(z2, 0)
        r = h2 @ w3 + b3 - y
        total += float(r @ r)
        dy = 2 * r / len(y)
        d2 = dy[:, None] * w3 * (z2 > 0)
        d1 = (d2 @ W2.T) * (z1 > 0)
        g = np.concatenate([(x.T @ d1).ravel(), d1.sum(0), (h1.T @ d2).ravel(), d2.sum(0), h2.T @ dy, [dy.sum()]])
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p - lr * (m / (1 - 0.9 ** (k + 1))) / (np.sqrt(v / (1 - 0.999 ** (k + 1))) + 1e-8)
    return total / len(t), p


def _split(p):
    W1, b1, W2, b2, w3, b3 = np.split(p, np.cumsum([24 * 64, 64, 64 * 64, 64, 64]))
    return W1.reshape(24, 64), b1, W2.reshape(64, 64), b2, w3, b3


def exact(case, seed):
    c = case
    if c["kind"] == "model":
        X, t, p, Xp = _samples(c, seed)
        loss, p = _epoch(X, t, p, c["batch"], 3e-3)
        W1, b1, W2, b2, w3, b3 = _split(p)
        y = np.maximum(np.maximum(Xp.astype(np.float64) @ W1 + b1, 0) @ W2 + b2, 0) @ w3 + b3
        return [np.array([loss]), p, y]
    if c["kind"] == "mine":
        if c["n"] * c["K"] > 2.5e6:
            return None
        ty, t, _ = _stream(c, seed, c["n"])
        unit = 1000 if c["ts"] == "i32" else 1000000
        by = _lists(ty.cpu().numpy(), t.cpu().numpy(), c["K"])
        levels = _levels(by, [(a * unit, b * unit) for a, b in MENU_MS], c["max_size"], c["threshold"])
        return levels and _patterns(c, [x[:2] for x in levels], {i + 1: x[2:] for i, x in enumerate(levels)})
    if _visits(c, busy=True) * (1 + c.get("chunks", 0)) > 1e8 or c.get("order"):
        return None
    if c["kind"] in ("query", "append"):
        n, k = c["n"], c.get("chunks", 0)
        ty, t, planted = _stream(c, seed, n + k * c.get("chunk", 0))
        ty, t, cands = ty.cpu().numpy(), t.cpu().numpy(), _candidates(c, seed, c["m"], planted)
        ends = [n + i * c.get("chunk", 0) for i in range(k + 1)]
        return [_counts(_lists(ty[:e], t[:e], c["K"]), cands) for e in ends]
    return [_counts(_lists(ty.cpu().numpy(), t.cpu().numpy(), c["K"]), cands) for ty, t, cands in _inputs(c, seed)]
