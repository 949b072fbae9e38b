"""Level-wise discovery counted with near rows (no end-event lists): every
level's candidates and counts equal the oracle's.  The inputs reach the edges
of the clusters that the rows count: entries far apart, clusters whose
occurrences all overlap, clusters of more entries than a wave has lanes, equal
times, one to eight intervals and types in one to three words of a row."""
import numpy as np
import pytest

import spikegen as sg
from oracle import apriori
from paper_0905_2203_amd import epi

pytestmark = pytest.mark.gpu


def poisson(seed, K, rate, dur, ts_kind, grid=1):
    unit = 1_000_000 if ts_kind else 1000
    s = sg.poisson_stream(np.random.Generator(np.random.PCG64(seed)), K=K, rate_hz=rate, dur_s=dur, ts_kind=ts_kind,
                          unit_per_ms=unit, cascades=[4], cascade_trigger_hz=[4.0])
    s["times"] = np.ascontiguousarray(s["times"] // grid * grid)
    return s


def bursts():
    # trains of 90 to 200 events a millisecond apart, of three types in turn, and lone cascades far from any other
    rng = np.random.Generator(np.random.PCG64(7))
    ty, t, at = [], [], 1000
    for b in range(24):
        n = int(rng.integers(90, 200))
        ty += [i % 3 for i in range(n)]
        t += [at + 1000 * i for i in range(n)]
        at = t[-1] + 300000
        for k in range(int(rng.integers(1, 40))):
            ty += [0, 1, 2, 3]
            t += [at, at + 2000, at + 4000, at + 9000]
            at += 100000
    return dict(types=np.asarray(ty, np.int32), times=np.asarray(t, np.int32), K=5, ts_kind=0)


CASES = {
    "sparse": (lambda: poisson(1, 40, 12.0, 20.0, 0), [(0, 5000), (5000, 10000), (10000, 20000)], 5, 10),
    "dense": (lambda: poisson(2, 5, 120.0, 6.0, 0), [(0, 5000), (5000, 20000)], 4, 50),
    "bursts": (bursts, [(0, 1000), (1000, 3000), (0, 30000)], 4, 30),
    "three_words_ns": (lambda: poisson(3, 130, 5.0, 20.0, 1), [(0, 9_000_000)], 4, 8),
    "two_words_menu8": (lambda: poisson(4, 66, 4.0, 20.0, 0), [(i * 2000, i * 2000 + 3000) for i in range(8)], 3, 4),
    "equal_times": (lambda: poisson(5, 9, 25.0, 15.0, 0, grid=4000),
                    [(0, 4000), (4000, 8000), (0, 12000), (3999, 20001)], 4, 25),
    "all_frequent": (lambda: poisson(6, 4, 5.0, 15.0, 1), [(0, 5_000_000), (5_000_000, 20_000_000)], 4, -1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_counts_by_near_rows(name):
    make, menu, size, theta = CASES[name]
    s = make()
    ref = apriori.mine(s, menu, size, theta)
    print(f"[gpu-near] {name}: n={s['types'].size} {[(len(r['counts']), len(r['frequent'])) for r in ref]}", flush=True)
    assert len(ref) >= 3
    with epi.Context(0) as ctx:
        ctx.epi_set_option(epi.EPI_OPT_MINE_LIST_ALPHAS, 0)
        sid = ctx.epi_load_stream(s["types"], s["times"], s["K"])
        for list_bytes in (8 << 30, 0):  # chain lists written in pieces and by one walk a parent
            ctx.epi_set_option(epi.EPI_OPT_MINE_LIST_BYTES, list_bytes)
            mid = ctx.epi_mine(sid, menu, size, theta)
            assert ctx.epi_mine_levels(mid) == len(ref)
            for L in range(2, len(ref) + 1):
                c, counts = ctx.epi_mine_read(mid, L)
                want = {(ty, tuple(menu[v] for v in iv)): n for (ty, iv), n in ref[L - 1]["counts"].items()}
                got = {(tuple(c["types"][i, :L].tolist()),
                        tuple(zip(c["lo"][i, : L - 1].tolist(), c["hi"][i, : L - 1].tolist()))): int(counts[i])
                       for i in range(c["N"].size)}
                assert got == want
            ctx.epi_mine_release(mid)
