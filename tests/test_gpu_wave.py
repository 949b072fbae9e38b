"""The wave chains (the counting kernels of the default engine) where they can go wrong, against the oracle: types
with as many events as a window takes and one more, single events, silences longer than a window may span, long
spans, lower bounds at the limit of what a chain list hands on and just beyond it (counted by the lane machines),
dense equal times, every size, segments, both timestamp kinds, batched, and appended events."""
import numpy as np
import pytest

import oracle
import spikegen as sg
from paper_0905_2203_amd import epi

pytestmark = pytest.mark.gpu
EVENTS = 256  # of one type in a window
GAP = 63      # a type's events i and i + 63 are at least the largest lower bound apart


def stream(types, times, kind):
    order = np.argsort(times, kind="stable")
    return dict(types=np.asarray(types, np.int32)[order], K=int(max(types)) + 1, ts_kind=kind,
                times=np.asarray(times, np.int64 if kind else np.int32)[order])


def per_type(rng, counts, period):
    """Each type's events at jittered multiples of its period, so that all types span the same time."""
    ty, t = [], []
    for k, n in enumerate(counts):
        step = period * max(counts) // max(n, 1)
        ty.append(np.full(n, k))
        t.append(np.arange(n) * step + rng.integers(0, max(1, step), size=n))
    return np.concatenate(ty), np.concatenate(t)


def episodes(rng, m, K, hi, sizes=(1, 8)):
    eps = []
    for _ in range(m):
        n = int(rng.integers(sizes[0], min(sizes[1], K) + 1))
        lo = rng.integers(0, hi // 2 + 1, size=n - 1)
        eps.append((rng.permutation(K)[:n], lo, lo + rng.integers(1, hi // 2 + 1, size=n - 1)))
    return sg.candidates_from_list(eps)


def least_gap(s):
    return min((int((t[GAP:] - t[:-GAP]).min()) for t in (s["times"][s["types"] == k].astype(np.int64) for k in range(s["K"]))
                if t.size > GAP), default=None)


def check(s, c, segments=(0, 1, 3), batched=True):
    want = oracle.count(s, c)
    with epi.Context(0) as ctx:
        sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
        cid = ctx.epi_submit_candidates(sid, c)
        for seg in segments:
            ctx.epi_set_option(epi.EPI_OPT_SEGMENTS, seg)
            ctx.epi_count([cid])
            got = ctx.epi_read_counts(cid, c["N"].size)
            assert np.array_equal(got, want), f"plain, segments {seg}: {np.flatnonzero(got != want)[:5]}"
            if batched:
                for sched in (epi.EPI_SCHED_RR, epi.EPI_SCHED_HEURISTIC):
                    ctx.epi_count([cid], epi.EPI_MODE_BATCHED, sched)
                    assert np.array_equal(ctx.epi_read_counts(cid, c["N"].size), want), f"batched {sched}, segments {seg}"
    return want


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, EVENTS - 1, EVENTS, EVENTS + 1, 2 * EVENTS, 2 * EVENTS + 1, 1500])
def test_events_per_type(n, kind):
    rng = np.random.default_rng(n + kind)
    counts = [n, max(1, n // 2), n, max(1, n // 7), n, 1, n, n, max(1, n - 1)]
    s = stream(*per_type(rng, counts, 1000), kind)
    check(s, episodes(rng, 120, s["K"], 6000))


def test_silences_and_long_spans():
    """Bursts separated by more than a window may span (2^30 units), spans up to just below 2^29, and chains that
    cross the silences (lower bounds of tens of millions)."""
    rng = np.random.default_rng(5)
    ty, t = [], []
    for b in range(12):
        n = 900
        ty.append(rng.integers(0, 9, size=n))
        t.append(b * (3 << 30) * (b % 3 + 1) + rng.integers(0, 400_000_000, size=n))
    s = stream(np.concatenate(ty), np.concatenate(t), 1)
    c = sg.concat_candidates(episodes(rng, 100, 9, 2_000_000), episodes(rng, 60, 9, 120_000_000, (2, 5)))
    want = check(s, c)
    assert want.max() > 50


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("over", [0, 1])
def test_lower_bound_at_the_hand_on_limit(kind, over):
    """A type's 64 events just fit the largest lower bound (over = 0), or are one unit too close (over = 1)."""
    rng = np.random.default_rng(8 + kind)
    s = stream(*per_type(rng, [4000, 3900, 4000, 2000], 40), kind)
    lo = least_gap(s) + over
    eps = [(rng.permutation(4)[:n], [lo] * (n - 1), [lo + w] * (n - 1)) for n in (2, 3, 4) for w in (1, 7, 40, 333, 5000)]
    # (bounds of at most 15 disjoint intervals only: deeper episodes are counted elsewhere)
    eps = [e for e in eps if 1 + e[2][0] // (e[2][0] - e[1][0] + 1) <= 15]
    want = check(s, sg.candidates_from_list(eps))
    assert want.max() > 20


@pytest.mark.parametrize("ties", [4, 60, 80])
def test_equal_times(ties):
    """Many events of a type at one time: below the wave chains' limit of 63, and above it."""
    rng = np.random.default_rng(ties)
    n = 6000
    s = stream(rng.integers(0, 5, size=n), rng.integers(0, n // (4 * ties), size=n) * 3, 0)
    check(s, episodes(rng, 80, 5, 8))


def test_appended_events():
    rng = np.random.default_rng(21)
    s = stream(*per_type(rng, [3000, 2500, 3000, 400, 3000, 1000], 500), 1)
    c = episodes(rng, 150, 6, 4000)
    n = s["types"].size
    cuts = [0, 1, n // 2, n // 2 + 1, n // 2 + 900, n]
    with epi.Context(0) as ctx:
        first = slice(0, cuts[2])
        sid = ctx.epi_load_stream(s["types"][first], s["times"][first], s["K"])
        cid = ctx.epi_submit_candidates(sid, c)
        ctx.epi_count([cid])
        for a, b in zip(cuts[2:-1], cuts[3:]):
            ctx.epi_append_stream(sid, s["types"][a:b], s["times"][a:b])
            ctx.epi_count([cid], epi.EPI_MODE_INCREMENTAL)
            part = dict(s, types=s["types"][:b], times=s["times"][:b])
            assert np.array_equal(ctx.epi_read_counts(cid, c["N"].size), oracle.count(part, c)), f"events 0..{b}"


@pytest.mark.parametrize("m,kind", [(64, 0), (65, 1), (300, 0)])
def test_skewed_episodes_in_listed_slots(m, kind):
    """Batched: few episodes have many segments and most have one, so the queue runs over a list of the slots at work;
    two sets of different streams, every schedule twice (the second from the kept plan)."""
    rng = np.random.Generator(np.random.PCG64(70 + m))
    sets, ctx = [], epi.Context(0)
    with ctx:
        for busy in (60000, 23000):
            types, times = per_type(rng, [busy] + [200] * 9, 50)
            s = stream(types, times, kind)
            eps = [(np.arange(1, 10)[rng.permutation(9)[:n]], np.zeros(n - 1, int), rng.integers(2000, 40000, size=n - 1))
                   for n in rng.integers(1, 5, size=m)]
            for i in rng.permutation(m)[:5]:  # with the busy type
                eps[i] = (np.concatenate([[0], eps[i][0]]), np.zeros(eps[i][0].size, int),
                          rng.integers(200, 40000, size=eps[i][0].size))
            c = sg.candidates_from_list(eps)
            sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
            sets.append((ctx.epi_submit_candidates(sid, c), c["N"].size, oracle.count(s, c)))
        for sched in (epi.EPI_SCHED_RR, epi.EPI_SCHED_HEURISTIC):
            for _ in range(2):
                ctx.epi_count([cid for cid, _, _ in sets], epi.EPI_MODE_BATCHED, sched)
                for cid, k, want in sets:
                    assert np.array_equal(ctx.epi_read_counts(cid, k), want)


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("over", [0, 1])
def test_lower_bound_of_127_events(kind, over):
    """Lists that hand on up to 128 entries: a type's 128 events just fit the largest lower bound, or do not by one unit
    (the lane machines then count); plain, batched, in segments, and appended to."""
    rng = np.random.default_rng(80 + kind)
    s = stream(*per_type(rng, [9000, 8700, 9000, 3000], 40), kind)
    times = [s["times"][s["types"] == k].astype(np.int64) for k in range(s["K"])]
    lo = min(int((t[127:] - t[:-127]).min()) for t in times) + over
    eps = [(rng.permutation(4)[:n], [lo] * (n - 1), [lo + w] * (n - 1)) for n in (2, 3, 4) for w in (333, 700, 5000)]
    eps = [e for e in eps if 1 + e[2][0] // (e[2][0] - e[1][0] + 1) <= 15]
    c = sg.candidates_from_list(eps)
    assert check(s, c).max() > 20
    n = s["types"].size
    with epi.Context(0) as ctx:
        sid = ctx.epi_load_stream(s["types"][: n - 700], s["times"][: n - 700], s["K"])
        cid = ctx.epi_submit_candidates(sid, c)
        ctx.epi_count([cid])
        for a, b in ((n - 700, n - 699), (n - 699, n)):
            ctx.epi_append_stream(sid, s["types"][a:b], s["times"][a:b])
            ctx.epi_count([cid], epi.EPI_MODE_INCREMENTAL)
        assert np.array_equal(ctx.epi_read_counts(cid, c["N"].size), oracle.count(s, c))
