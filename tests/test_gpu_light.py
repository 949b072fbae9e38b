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


@pytest.mark.parametrize("m,kind", [(1, 0), (63, 1), (5000, 0), (70001, 1), (300007, 0)])
def test_light_slots_in_runs(m, kind):
    rng = np.random.default_rng(m)
    s = stream(700, 24, kind, m)
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
