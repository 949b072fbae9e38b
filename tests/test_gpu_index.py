"""The stream index at the edges of its tiles (256 to 4096 events, four waves each), types from one to the most a
stream may have: the per-type index equals a stable sort by type, and the tile-major copy (read by the state
machines, which count with a work log) gives the oracle's counts.  Host, device and appended events."""
import numpy as np
import pytest
import torch

import oracle
import spikegen as sg
from paper_0905_2203_amd import epi

pytestmark = pytest.mark.gpu


def make(rng, n, K, kind, step):
    times = np.cumsum(rng.integers(0, 2 * step + 1, size=n))
    return dict(types=rng.integers(0, K, size=n).astype(np.int32), K=K, ts_kind=kind,
                times=times.astype(np.int64 if kind else np.int32))


def check(ctx, sid, s):
    off, ts = ctx.epi_read_type_index(sid)
    order = np.argsort(s["types"], kind="stable")
    assert np.array_equal(off, np.searchsorted(s["types"][order], np.arange(s["K"] + 1)))
    assert np.array_equal(ts, s["times"][order])
    if s["K"] < 3:
        return
    present = np.unique(s["types"])
    rng = np.random.default_rng(1)
    eps = []
    for _ in range(40):
        ty = rng.permutation(present)[: int(rng.integers(1, min(4, present.size) + 1))]
        lo = rng.integers(0, 20, size=ty.size - 1)
        eps.append((ty, lo, lo + rng.integers(10, 400, size=ty.size - 1)))
    c = sg.candidates_from_list(eps)
    cid = ctx.epi_submit_candidates(sid, c)
    ctx.epi_set_option(epi.EPI_OPT_WORKLOG, 1)
    ctx.epi_count([cid])
    got = ctx.epi_read_counts(cid, c["N"].size)
    ctx.epi_set_option(epi.EPI_OPT_WORKLOG, 0)
    ctx.epi_release_set(cid)
    assert np.array_equal(got, oracle.count(s, c))


@pytest.mark.parametrize("K", [1, 2, 3, 64, 65, 255, 256, 257, 4096])
@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 2047, 2048, 2049, 4097, 70001])
def test_index(n, K):
    rng = np.random.default_rng(n + K)
    kind = (n + K) % 2
    # (every other one so sparse that the stream picks its smallest tiles)
    s = make(rng, n, K, kind, 3 if n % 2 or not kind else 1_500_000)
    with epi.Context(0) as ctx:
        check(ctx, ctx.epi_load_stream(s["types"], s["times"], K), s)
        d = [torch.from_numpy(s[k]).cuda() for k in ("types", "times")]
        torch.cuda.synchronize()
        check(ctx, ctx.epi_load_stream_device(d[0], d[1], K), s)
        cut = n // 3
        part = ctx.epi_load_stream(s["types"][:cut], s["times"][:cut], K)
        ctx.epi_append_stream(part, s["types"][cut:], s["times"][cut:])
        check(ctx, part, s)


def test_blocks_of_released_streams_and_sets():
    """Streams and sets of changing sizes loaded, counted on another stream and released in turn: the device memory
    they leave to the next ones is not in use any more."""
    rng = np.random.default_rng(2)
    side = torch.cuda.Stream()
    with epi.Context(0) as ctx:
        for i in range(12):
            n, K = int(rng.integers(500, 60000)), int(rng.integers(4, 40))
            s = make(rng, n, K, i % 2, 5)
            c = sg.random_candidates(rng, int(rng.integers(50, 900)), K, 1, 4, 3)
            d = [torch.from_numpy(s[k]).cuda() for k in ("types", "times")]
            torch.cuda.synchronize()
            sid = (ctx.epi_load_stream_device(d[0], d[1], K, side.cuda_stream) if i % 3 else
                   ctx.epi_load_stream(s["types"], s["times"], K))
            cid = ctx.epi_submit_candidates(sid, c)
            ctx.epi_count([cid], hip_stream=side.cuda_stream if i % 4 else None)
            if i % 2:
                got = ctx.epi_read_counts(cid, c["N"].size)
                assert np.array_equal(got, oracle.count(s, c)), i
            ctx.epi_release_set(cid)  # (the even rounds' counts still run)
            ctx.epi_release_stream(sid)
