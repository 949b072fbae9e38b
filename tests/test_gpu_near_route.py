"""Which way a level of 512 and more parents is counted: by near rows, or, where one wave would walk a cluster long
after the others, by lists.  The premise (the longest cluster's share of all positions) is computed here for the
parents' chain lists, and every level's counts equal the oracle's on both sides of the rule."""
import numpy as np
import pytest

from oracle import apriori
from paper_0905_2203_amd import epi

pytestmark = pytest.mark.gpu
MENU = [(0, 4000), (4000, 9000), (9000, 20000)]
H, LONE, LEAST, K = 20000, 1500, 2048, 16


def stream(busy, seed):
    """K quiet types over 60 s, and, if busy, two of them at 600 Hz beside."""
    rng = np.random.default_rng(seed)
    t = [rng.integers(1, 60_000_000, size=5000)] + [rng.integers(1, 60_000_000, size=70000)] * busy
    ty = [rng.integers(0, K, size=5000)] + [rng.integers(0, 2, size=70000)] * busy
    t, ty = np.concatenate(t), np.concatenate(ty)
    order = np.argsort(t, kind="stable")
    return dict(types=ty[order].astype(np.int32), times=t[order].astype(np.int32), K=K, ts_kind=0)


def clusters(s, pairs):
    """(longest, all): stream positions from first to last entry of the clusters of the pairs' chain lists, a window after each."""
    pos = [np.flatnonzero(s["types"] == k) for k in range(K)]
    n = s["times"].size
    window = n * H / float(int(s["times"][-1]) - int(s["times"][0]))
    longest, total = 0, 0.0
    for (a, b), (lo, hi) in pairs:
        ta, tb = s["times"][pos[a]].astype(np.int64), s["times"][pos[b]].astype(np.int64)
        i = np.searchsorted(ta, tb - lo, side="left") - 1
        ok = (i >= 0) & (tb - ta[np.maximum(i, 0)] <= hi)
        e, st, p = tb[ok], ta[i[ok]], pos[b][ok]
        head = np.concatenate([[True], st[1:] > e[:-1] + H])
        first = np.flatnonzero(head)
        last = np.concatenate([first[1:] - 1, [len(p) - 1]])
        span = p[last] - p[first]
        longest, total = max(longest, int(span.max())), total + float(span.sum()) + window * len(first)
    return longest, total


@pytest.mark.parametrize("busy", [0, 1])
def test_route_by_the_longest_cluster(busy):
    s = stream(busy, 4 + busy)
    theta = 5
    ref = apriori.mine(s, MENU, 3, theta)
    pairs = [(ty, MENU[iv[0]]) for ty, iv in ref[1]["frequent"]]
    longest, total = clusters(s, pairs)
    print(f"[gpu-near-route] busy={busy}: {len(pairs)} parents, longest {longest} of {total:.0f}", flush=True)
    assert len(pairs) >= 512
    assert (longest >= LEAST and longest * LONE > total) == bool(busy)
    with epi.Context(0) as ctx:
        sid = ctx.epi_load_stream(s["types"], s["times"], K)
        for list_bytes in (8 << 30, 0):  # with lists, and one walk a parent where lists may not be kept
            ctx.epi_set_option(epi.EPI_OPT_MINE_LIST_BYTES, list_bytes)
            mid = ctx.epi_mine(sid, MENU, 3, theta)
            assert ctx.epi_mine_levels(mid) == len(ref)
            for L in range(2, len(ref) + 1):
                c, counts = ctx.epi_mine_read(mid, L)
                want = {(ty, tuple(MENU[v] for v in iv)): n for (ty, iv), n in ref[L - 1]["counts"].items()}
                got = {(tuple(c["types"][i, :L].tolist()),
                        tuple(zip(c["lo"][i, : L - 1].tolist(), c["hi"][i, : L - 1].tolist()))): int(counts[i])
                       for i in range(c["N"].size)}
                assert got == want
            ctx.epi_mine_release(mid)


def test_bytes_of_a_level_counted_by_rows():
    """epi_mine_level_bytes of such a level: the entries and the rows they read, the positions of the windows that are
    walked (clusters with two occurrences that do not overlap), and the counts."""
    s = stream(0, 4)
    theta, M = 5, len(MENU)
    ref = apriori.mine(s, MENU, 3, theta)
    frequent = set(ref[1]["frequent"])
    starts = {}
    for (a, b), iv in frequent:
        starts.setdefault(a, []).append(b)
    t = s["times"].astype(np.int64)
    pos = [np.flatnonzero(s["types"] == k) for k in range(K)]
    wend = np.searchsorted(t, t + H, side="right")
    entries = rows = walked = 0
    for (a, b), iv in frequent:
        lo, hi = MENU[iv[0]]
        ta, tb = t[pos[a]], t[pos[b]]
        i = np.searchsorted(ta, tb - lo, side="left") - 1
        ok = (i >= 0) & (tb - ta[np.maximum(i, 0)] <= hi)
        e, st, p = tb[ok], ta[i[ok]], pos[b][ok]
        entries += e.size
        if not any(c != a for c in starts.get(b, [])):
            continue  # no extension: nothing is counted
        rows += e.size * (M + 1)
        first = np.flatnonzero(np.concatenate([[True], st[1:] > e[:-1] + H]))
        for f, l in zip(first, np.concatenate([first[1:], [e.size]])):
            if st[l - 1] > e[f]:  # not simple
                covered = 0
                for j in range(f, l):
                    walked += max(0, wend[p[j]] - max(p[j] + 1, covered))
                    covered = max(covered, wend[p[j]])
    assert walked > 0
    with epi.Context(0) as ctx:
        sid = ctx.epi_load_stream(s["types"], s["times"], K)
        mid = ctx.epi_mine(sid, MENU, 3, theta)
        m = ctx.epi_mine_level_info(mid, 3)[0]
        assert m == len(ref[2]["counts"])
        assert ctx.epi_mine_level_bytes(mid, 3) == walked * (2 + 4) + entries * 12 + rows * 8 + m * 4
