"""The engines behind the wave chains, each against the oracle where the chains are refused.

The chains take every stream whose types have no 128 events within a lower bound, so the tests of the other engines
meet them by default.  Here a type with 128 events at one time (in the stream, and in one episode of each size)
refuses them: the lane machines count, with packed and separate keys, plain in segments, batched, incrementally, and
in one batched plan beside chains.  EPI_OPT_LANE_ENGINE = 0 refuses them too: the LDS machines count at the bounds of
their relative times, and the per-event tracking engine in time order."""
import numpy as np
import pytest

import oracle
import spikegen as sg
import test_gpu_lane as lane
import test_gpu_relative_times as relative
import test_gpu_tracking as tracking
from paper_0905_2203_amd import epi

pytestmark = pytest.mark.gpu
TIES = 128


@pytest.fixture(scope="module")
def ctx():
    c = epi.Context(0)
    yield c
    c.close()


@pytest.fixture
def machines(ctx):
    ctx.epi_set_option(epi.EPI_OPT_LANE_ENGINE, 0)
    yield ctx
    ctx.epi_set_option(epi.EPI_OPT_LANE_ENGINE, 1)


def with_ties(s):
    """The stream with one more type, whose TIES events share the time of the middle event."""
    i = s["times"].size // 2
    return dict(s, K=s["K"] + 1, types=np.insert(s["types"], [i] * TIES, s["K"]).astype(np.int32),
                times=np.insert(s["times"], [i] * TIES, s["times"][i]).astype(s["times"].dtype))


def tied_episodes(s, unit):
    """An episode of each size with the type of the ties."""
    K, eps = s["K"] - 1, []
    for n in range(1, min(8, K) + 1):
        ty = list(range(n))
        ty[n // 2] = K
        eps.append((ty, [0] * (n - 1), [10 * unit] * (n - 1)))
    return sg.candidates_from_list(eps)


@pytest.mark.parametrize("name", ["int32_us", "int64_ns_dense", "int64_ns_bursty", "int64_ns_sparse", "int64_ns_29bit"])
def test_lane_machines(ctx, name):
    s = with_ties(dict(lane._streams())[name])
    unit = s["unit_per_ms"]
    if name == "int64_ns_29bit":
        # 512-event tiles are too long for the packed keys, 256-event tiles fit them from 2^28 ns on
        assert lane._longest_tile(s["times"], 512) >= (1 << 29) - 1
        assert (1 << 28) <= lane._longest_tile(s["times"], 256) < (1 << 29) - 1
    rng = np.random.Generator(np.random.PCG64(61))
    c = sg.concat_candidates(lane._episodes(rng, s["K"] - 1, unit, 400), tied_episodes(s, unit))
    m = c["N"].size
    want = oracle.count(s, c)
    assert want.max() > 50
    sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
    cid = ctx.epi_submit_candidates(sid, c)
    try:
        for seg in (1, 3, 17, 0):
            ctx.epi_set_option(epi.EPI_OPT_SEGMENTS, seg)
            for mode, sched in ((epi.EPI_MODE_PLAIN, epi.EPI_SCHED_RR), (epi.EPI_MODE_BATCHED, epi.EPI_SCHED_RR),
                                (epi.EPI_MODE_BATCHED, epi.EPI_SCHED_HEURISTIC)):
                got = lane._count(ctx, cid, m, mode, sched)
                assert np.array_equal(got, want), f"segments {seg} mode {mode}: {np.flatnonzero(got != want)[:5]}"
    finally:
        ctx.epi_set_option(epi.EPI_OPT_SEGMENTS, 0)
        ctx.epi_release_set(cid)
        ctx.epi_release_stream(sid)


@pytest.mark.parametrize("kind", [0, 1])
def test_lane_machines_on_appended_events(ctx, kind):
    unit = 1_000_000 if kind else 1000
    rng = np.random.Generator(np.random.PCG64(62 + kind))
    s = with_ties(sg.poisson_stream(rng, K=9, rate_hz=30.0, dur_s=30.0, ts_kind=kind, unit_per_ms=unit))
    c = sg.concat_candidates(lane._episodes(rng, 9, unit, 150), tied_episodes(s, unit))
    m, n = c["N"].size, s["types"].size
    cuts = [n // 2 - 300, n // 2 + 40, n // 2 + 41, n]  # (the first cut before the ties, the second among them)
    sid = ctx.epi_load_stream(s["types"][:cuts[0]], s["times"][:cuts[0]], s["K"])
    cid = ctx.epi_submit_candidates(sid, c)
    ctx.epi_count([cid])
    for a, b in zip(cuts, cuts[1:]):
        ctx.epi_append_stream(sid, s["types"][a:b], s["times"][a:b])
        ctx.epi_count([cid], epi.EPI_MODE_INCREMENTAL)
        part = dict(s, types=s["types"][:b], times=s["times"][:b])
        assert np.array_equal(ctx.epi_read_counts(cid, m), oracle.count(part, c)), f"events 0..{b}"
    ctx.epi_release_set(cid)
    ctx.epi_release_stream(sid)


def test_chains_and_lane_machines_in_one_plan(ctx):
    rng = np.random.Generator(np.random.PCG64(64))
    plain = sg.poisson_stream(rng, K=10, rate_hz=30.0, dur_s=40.0, ts_kind=1, unit_per_ms=1_000_000)
    sets = []
    for s in (plain, with_ties(plain)):
        c = lane._episodes(rng, 10, 1_000_000, 300)
        sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
        sets.append((ctx.epi_submit_candidates(sid, c), c["N"].size, oracle.count(s, c)))
    for seg in (0, 5):
        ctx.epi_set_option(epi.EPI_OPT_SEGMENTS, seg)
        for sched in (epi.EPI_SCHED_RR, epi.EPI_SCHED_HEURISTIC):
            for _ in range(2):  # (the second from the kept plan)
                ctx.epi_count([cid for cid, _, _ in sets], epi.EPI_MODE_BATCHED, sched)
                for cid, m, want in sets:
                    assert np.array_equal(ctx.epi_read_counts(cid, m), want)
    ctx.epi_set_option(epi.EPI_OPT_SEGMENTS, 0)


def test_relative_times_at_the_bound(machines):
    relative.test_relative_times_at_the_bound(machines)


def test_int64_machines_beyond_the_bound(machines):
    relative.test_int64_machines_beyond_the_bound(machines)


@pytest.mark.parametrize("kind", [0, 1])
def test_tracking_engine_long_episodes(machines, kind):
    tracking.test_tracking_long_episodes(machines, kind)


def test_tracking_engine_equal_times(machines):
    tracking.test_tracking_equal_times(machines)


def test_tracking_engine_repeated_types(machines):
    tracking.test_tracking_repeated_types(machines)


def test_tracking_engine_heavy_type(machines):
    """2.4 million events of a type: more than 1024 compaction blocks, 22 pointer-jumping rounds."""
    tracking.test_tracking_heavy_type_and_empty_set(machines)


def test_tracking_engine_then_incremental(machines):
    tracking.test_tracking_then_incremental(machines)
