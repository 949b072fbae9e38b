"""Very many light episodes, whose slots the waves of a batched count take in runs: fewer slots than a run, a run more
or less than the waves share out, a stretch of skewed ones among them; every count equals the oracle's."""
import numpy as np
import pytest

import oracle
import spikegen as sg
from paper_0905_2203_amd import epi

pytestmark = pytest.mark.gpu


def stream(n, K, kind, seed):
    rng = np.random.default_rng(seed)
    t = np.sort(rng.integers(0, 2000 * n, size=n))
    return dict(types=rng.integers(0, K, size=n).astype(np.int32), times=t.astype(np.int64 if kind else np.int32), K=K, ts_kind=kind)


def episodes(rng, m, K, hi):
    N = rng.integers(1, 4, size=m)
    live = np.arange(7)[None, :] < N[:, None] - 1
    lo = np.where(live, rng.integers(0, hi // 4, size=(m, 7)), 0)
    ty = np.argsort(rng.random((m, K)), axis=1)[:, :8]
    return dict(N=N.astype(np.uint8), types=np.where(np.arange(8)[None, :] < N[:, None], ty, -1).astype(np.int32), lo=lo.astype(np.int64),
                hi=np.where(live, lo + rng.integers(hi // 4, hi, size=(m, 7)), 0).astype(np.int64))


@pytest.mark.parametrize("m,n,kind", [(1, 700, 0), (63, 700, 1), (5000, 700, 0), (70001, 700, 1), (300007, 1600, 0)])
def test_light_slots_in_runs(m, n, kind):
    rng = np.random.default_rng(m)
    s = stream(n, 24, kind, m)
    c = episodes(rng, m, 24, 60000)
    want = oracle.count(s, c)
    with epi.Context(0) as ctx:
        sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
        cid = ctx.epi_submit_candidates(sid, c)
        for sched in (epi.EPI_SCHED_RR, epi.EPI_SCHED_HEURISTIC):
            ctx.epi_count([cid], epi.EPI_MODE_BATCHED, sched)
            assert np.array_equal(ctx.epi_read_counts(cid, m), want)


def test_light_and_heavy_sets_together():
    """A few segmented episodes of a long stream beside very many of a short one."""
    rng = np.random.default_rng(3)
    sets = []
    with epi.Context(0) as ctx:
        for n, m in ((120000, 40), (500, 60000)):
            s = stream(n, 20, 1, n)
            c = episodes(rng, m, 20, 60000)
            sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
            sets.append((ctx.epi_submit_candidates(sid, c), m, oracle.count(s, c)))
        for _ in range(2):
            ctx.epi_count([cid for cid, _, _ in sets], epi.EPI_MODE_BATCHED, epi.EPI_SCHED_RR)
            for cid, m, want in sets:
                assert np.array_equal(ctx.epi_read_counts(cid, m), want)


@pytest.mark.parametrize("m,n", [(1 << 18, 500), ((1 << 19) + 3, 100)])
def test_very_many_episodes_of_a_few_events(m, n):
    """Counted by the machines (64 episodes a wave): batched at most 64 events an episode, plain at most 16."""
    rng = np.random.default_rng(n)
    s = stream(n, 24, 0, n)
    c = episodes(rng, m, 24, 60000)
    events = np.bincount(s["types"], minlength=24)
    per = sum(np.where(c["types"][:, k] >= 0, events[c["types"][:, k]], 0) for k in range(8))
    assert per.mean() < (64 if n == 500 else 16)
    want = oracle.count(s, c)
    with epi.Context(0) as ctx:
        sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
        cid = ctx.epi_submit_candidates(sid, c)
        for mode in (epi.EPI_MODE_PLAIN, epi.EPI_MODE_BATCHED):
            ctx.epi_count([cid], mode)
            assert np.array_equal(ctx.epi_read_counts(cid, m), want)


@pytest.mark.parametrize("per_cell", [0.7, 3.0])
def test_events_far_apart(per_cell):
    """int64 streams whose windows hold fewer or more events of a type than the chains need (1.4): plain, batched,
    tracking, and appended to across many windows."""
    rng = np.random.default_rng(int(per_cell * 10))
    n, K = 6000, 10
    t = np.sort(rng.integers(0, int(n / K / per_cell * (1 << 34)), size=n))
    t[1::2] = t[::2] + rng.integers(0, 400_000_000, size=n // 2)  # (half of them follow another closely)
    order = np.argsort(t, kind="stable")
    s = dict(types=rng.integers(0, K, size=n).astype(np.int32)[order], times=t[order].astype(np.int64), K=K, ts_kind=1)
    c = episodes(rng, 200, K, 170_000_000)
    cells = 1 + int((np.diff(s["times"] >> 34) != 0).sum())
    assert cells >= 64 and (n / K < 1.4 * cells) == (per_cell < 1)
    want = oracle.count(s, c)
    assert want.max() > 20
    with epi.Context(0) as ctx:
        sid = ctx.epi_load_stream(s["types"], s["times"], K)
        cid = ctx.epi_submit_candidates(sid, c)
        for mode in (epi.EPI_MODE_PLAIN, epi.EPI_MODE_BATCHED, epi.EPI_MODE_TRACKING):
            ctx.epi_count([cid], mode)
            assert np.array_equal(ctx.epi_read_counts(cid, 200), want)
        sid = ctx.epi_load_stream(s["types"][:n // 2], s["times"][:n // 2], K)
        cid = ctx.epi_submit_candidates(sid, c)
        ctx.epi_count([cid])
        ctx.epi_append_stream(sid, s["types"][n // 2:], s["times"][n // 2:])
        ctx.epi_count([cid], epi.EPI_MODE_INCREMENTAL)
        assert np.array_equal(ctx.epi_read_counts(cid, 200), want)
        ctx.epi_count([cid])
        assert np.array_equal(ctx.epi_read_counts(cid, 200), want)
