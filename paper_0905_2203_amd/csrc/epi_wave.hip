// Wave chains: the count of one candidate episode over a range of time by one
// 64-lane wave, parallel over the events of each node's type.
//
// For episode alpha and node k, the chain events are the events x of type
// alpha[k] that end an occurrence of alpha[1..k]; L_k(x) is the latest start of
// such an occurrence (L_1(x) = t_x).  Along a node's chain events L_k is
// non-decreasing, so the best predecessor of x is the latest chain event y of
// node k-1 with t_y < t_x - lo (if t_x <= t_y + hi): one binary search per
// event (Sec. IV-C), and only the chain events go on to the next node
// (Sec. IV-D/E).  The count is the greedy of Alg. 1 over the last node's
// (L_N(x), t_x): the next kept event is the first with L > the last kept one's
// time.  These are the completions of the serial state machine (Sec. III-A with
// starts admitted only strictly after the last completion), so segments, their
// records and the reconciliation are those of epi_tiled.hip.
//
// The wave walks time in windows.  A window starts at the earliest next event
// of the episode's types and ends where some type would have more than kCap
// events in it, so every node's events fit R registers a lane.  Node by node,
// the lanes read the node's events (coalesced, from the per-type index), search
// the previous node's chain list in LDS (R independent searches a lane in
// lockstep), and append the hits in time order.  From one window to the next a
// list hands on the entries a later event can still reach: those less than lo
// before the window's end, and the latest one before them (any other is
// dominated); that is at most 64 when the type has no 64 events within lo, at
// most 128 when it has no 128 (wave_hand, properties of the stream that the host
// checks).  The kernels that hand on 128 (HC = 2, in 64s) take 13.3 KB of LDS a
// wave instead of 8.7, so 12 waves a CU instead of 18: they count streams with
// such busy types alone (skewed rates, some 6 kHz in all and more).
//
// What bounds it: instruction issue and LDS latency.  A state machine lane
// takes its events one at a time (135 VALU instructions over the loop's paths,
// nearly all issued by a diverged wave, 64 events a pass); here a wave spends
// about 46 VALU and 36 SALU instructions on 64 events of a node, whatever the
// events do, and needs no tile staging, rings or rebasing.  80k episodes of 2-8
// nodes over 20M events of 256 types: 198 -> 50 ms (VALU issue 0.73; the index
// comes at 5 TB/s from beyond L2: cutting time so that a stretch stays in L2 gained
// nothing); 5k episodes of 1-6 nodes over 1.5M events: 24.8 -> 0.50 ms; 992 pairs
// over 10k events: 2.7 ms -> 53 us (a lane each had left the chip idle).
#include <algorithm>
#include <type_traits>

#include "epi_count.h"

namespace epi {

namespace {

constexpr int kW = 64;
constexpr int kR = kWaveChunks;
constexpr int kCap = kR * kW;
constexpr int kRunMin = 6;            // hits of 64 from which the greedy takes runs at a time

// Chain lists.  An entry is one 64-bit word, a time above the latest start of an
// occurrence ending there, so that one LDS access moves both.  int32 times: the
// two times themselves.  int64 times: the time from the window's first event
// (signed, 35 bits) above the start's low 29 bits (it is less than 2^29 before),
// so that one compare orders entries by time; 8 bytes an entry instead of 12 let
// a CU hold 18 waves instead of 14.  Entry 0 is a sentinel before every time: a
// search always ends on an entry.
template <typename T>
struct Entry {
    static constexpr bool kRel = sizeof(T) == 8;  // times from the window's first event
    static constexpr int kLow = kRel ? 29 : 32;
    static constexpr uint64_t kSpan = (uint64_t(1) << (63 - kLow)) - 1;  // longest window
    static_assert(!kRel || 63 - kLow == kCellBits, "cells of a stream are windows' spans");
    using Key = std::conditional_t<kRel, int64_t, int32_t>;   // what a search compares
    using UKey = std::make_unsigned_t<Key>;
    static constexpr int kKeyAt = kRel ? 0 : 4;               // byte of it in the entry
    static constexpr int kUp = kRel ? kLow : 0;               // a time's shift in a key
    static __device__ __forceinline__ Key key(T v, T h) {
        if constexpr (kRel) return (Key)(((uint64_t)v - (uint64_t)h) << kLow);
        else return v;
    }
    static __device__ __forceinline__ UKey len(int t) { return (UKey)(uint32_t)t << kUp; }
    static __device__ __forceinline__ int64_t make(Key k, uint32_t start) {
        if constexpr (kRel) return k | (int64_t)start;
        else return (int64_t)(((uint64_t)(uint32_t)k << 32) | start);
    }
    static __device__ __forceinline__ UKey key_of(int64_t e) {  // (with the start bits below it)
        return kRel ? (UKey)e : (UKey)((uint64_t)e >> 32);
    }
    static __device__ __forceinline__ uint32_t start_bits(T v) { return (uint32_t)v & (kRel ? (1u << 29) - 1 : ~0u); }
    static __device__ __forceinline__ T start(T v, uint32_t bits) {
        if constexpr (kRel) return (T)((uint64_t)v - (uint64_t)(((uint32_t)v - bits) & ((1u << 29) - 1)));
        else return (T)bits;
    }
};
template <int HC>
struct WaveLds {
    static constexpr int kHand = HC * kW;
    int64_t e[2][1 + kCap + kHand];  // a sentinel, handed-on entries, a window's events
    int64_t c[kMaxN - 1][kHand];     // handed on per node
};

// One candidate's episode as the wave holds it: lane k keeps node k's next
// index position and end, and interval k (between nodes k and k+1).
template <typename T>
struct WaveEp {
    int N;
    int32_t cur, end;
    int32_t lo, hi;
    T H;  // longest span
    int32_t P;  // its segments
    int64_t S;  // tiles each
};

__device__ __forceinline__ int rdlane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ int bcast(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t bcast(int64_t v) {
    const uint32_t a = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)b << 32) | a);
}
__device__ __forceinline__ int64_t rdlane(int64_t v, int l) {
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)b << 32) | a);
}
__device__ __forceinline__ int below(uint64_t m, int base) {  // base + set bits of m below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)base));
}
// The stream's times as global memory: a pointer read from a unit in memory
// would else make flat loads, which also count as LDS operations, so that every
// wait for a search would wait for the next node's events too.
template <typename T>
using Times = const __attribute__((address_space(1))) T *;
// the first n lanes
__device__ __forceinline__ uint64_t lanes_below(int n) {
    return n >= kW ? ~uint64_t(0) : n <= 0 ? 0 : (uint64_t(1) << n) - 1;
}
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// LDS operations of a wave complete in order; this only keeps the compiler
// from moving one lane's read before another lane's write.
__device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// All lanes meet here after one lane's stores: without it the compiler may send
// the other lanes into a loop's next round on their own (it knows that they
// skip every lane-0 branch), where they would read a queue position that only
// lane 0 fetches.
__device__ __forceinline__ void rejoin() { __builtin_amdgcn_wave_barrier(); }

// Segments of an episode whose types have `cost` events, and tiles each: by its
// own events, so that light episodes are not cut into pieces that cost more to
// start and reconcile than to count.
template <typename T>
__device__ __forceinline__ void own_segments(const CountArgs<T> &a, int64_t cost, int32_t &P, int64_t &S) {
    P = a.P;
    S = a.S;
    if (a.P > 1 && a.seg_cost > 0) {
        const int64_t want = cost / a.seg_cost + 1;
        const int32_t B = (int32_t)a.B, p = want < a.P ? (int32_t)want : a.P;
        S = (B + p - 1) / p;
        P = (B + (int32_t)S - 1) / (int32_t)S;
    }
}

template <typename T>
__device__ __forceinline__ WaveEp<T> load_episode(const CountArgs<T> &a, int64_t slot, int lane) {
    WaveEp<T> ep;
    ep.N = bcast((int)a.cN[slot]);
    ep.cur = ep.end = 0;
    ep.lo = ep.hi = 0;
    if (lane < ep.N) {
        const int32_t ty = a.ctypes[(int64_t)lane * a.m + slot];
        ep.cur = a.type_off[ty];
        ep.end = a.type_off[ty + 1];
    }
    if (lane + 1 < ep.N) {
        ep.lo = (int32_t)a.clo[(int64_t)lane * a.m + slot];
        ep.hi = (int32_t)a.chi[(int64_t)lane * a.m + slot];
    }
    int h = ep.hi;  // the span is below 2^29
    for (int d = 1; d < 8; d <<= 1) h += __shfl_xor(h, d, 8);
    ep.H = (T)bcast(h);
    int64_t c = ep.end - ep.cur;
    for (int d = 1; d < 8; d <<= 1) c += __shfl_xor(c, d, 8);
    own_segments(a, bcast(c), ep.P, ep.S);
    ep.P = bcast(ep.P);
    ep.S = bcast(ep.S);
    return ep;
}

// Move every node's position to its first event after time x: eight lanes a
// node, 9-ary search (six dependent loads for 200k events instead of eighteen).
template <typename T>
__device__ __forceinline__ void seek(Times<T> ts, WaveEp<T> &ep, T x, int lane) {
    const int node = lane >> 3, sub = lane & 7;
    int32_t lo = __shfl(ep.cur, node, kW), hi = __shfl(ep.end, node, kW);
    while (__ballot(lo < hi)) {
        const int32_t len = hi - lo;
        const int32_t at = lo + (int32_t)(((int64_t)len * (sub + 1)) / 9);  // < hi when len > 0
        const bool le = len > 0 && ts[at] <= x;
        const int c = __popc((uint32_t)(__ballot(le) >> (node * 8)) & 0xffu);  // pivots at or before x
        const int32_t nlo = c > 0 ? lo + (int32_t)(((int64_t)len * c) / 9) + 1 : lo;
        const int32_t nhi = c < 8 ? lo + (int32_t)(((int64_t)len * (c + 1)) / 9) : hi;
        if (len > 0) {
            lo = nlo;
            hi = nhi < nlo ? nlo : nhi;
        }
    }
    const int32_t v = __shfl(lo, (lane & 7) * 8, kW);
    if (lane < ep.N) ep.cur = v;
}

template <int NR>
using Chunks = std::integral_constant<int, NR>;

// Node k's next kCap events into x (the index is padded by kCap entries);
// returns how many its type has left.
template <typename T>
__device__ __forceinline__ int load_events(Times<T> ts, const WaveEp<T> &ep, int k, int lane, T (&x)[kR]) {
    const int c = rdlane(ep.cur, k);
    Times<T> p = ts + c;
#pragma unroll
    for (int r = 0; r < kR; ++r) x[r] = p[r * kW + lane];
    return rdlane(ep.end, k) - c;
}

// Every node's next event, and the one kCap after it (lane k: node k; lanes past
// the last node and types with fewer left read something in the padded index).
template <typename T>
__device__ __forceinline__ void load_heads(Times<T> ts, const WaveEp<T> &ep, T &h, T &f) {
    h = ts[ep.cur];
    f = ts[(int64_t)ep.cur + (ep.end - ep.cur > kCap ? kCap : 0)];
}

// What a run hands back, and what it is checked against.
template <typename T>
struct WaveOut {
    int32_t cnt = 0;   // completions at or after Bp
    T last;            // the last of them (unset when none)
    bool synced = false;
};
// The record of a segment's speculative run that a re-run may meet.
template <typename T>
struct WaveRec {
    int32_t c = 0;       // its completions
    T first[kRecFirst];  // the first of them
    T sync_t;            // Bp + H
};

// Count the completions of the episode over the events from its positions on
// and before Ep, given the last completion e0 (type minimum: none); every event
// from the positions on is after e0.  SYNC: a re-run that stops where it meets
// the speculative record (see rerun_segment in epi_tiled.hip); out.cnt then
// includes the record's remaining completions.
template <typename T, bool SYNC, int HC>
__device__ __forceinline__ void wave_run(Times<T> ts, WaveLds<HC> &w, WaveEp<T> &ep, T e0, T Bp, T Ep,
                                         int lane, T *__restrict__ first_out, int64_t first_stride,
                                         const WaveRec<T> *rec, WaveOut<T> &out) {
    using U = std::make_unsigned_t<T>;  // differences of ordered times: exact in it
    using E = Entry<T>;
    using Key = typename E::Key;
    using UKey = typename E::UKey;
    constexpr T kEnd = TsLimits<T>::hi();
    constexpr T kMin = TsLimits<T>::lo();
    const int N = ep.N;
    T tau = bcast(e0);
    T h0 = 0, te = 0;  // the window's first event and end
    if (lane < 2) w.e[lane][0] = INT64_MIN;
    lds_order();
    int nc = 0;  // lane k: entries node k's list handed on
    int32_t cnt = 0;
    // a window's first loads are issued in the one before it
    T hv, fv, x[kR];
    load_heads(ts, ep, hv, fv);
    int left = load_events(ts, ep, 0, lane, x);
    while (true) {
        T h = ep.cur < ep.end ? hv : kEnd, f = ep.end - ep.cur > kCap ? fv : kEnd;
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            const T oh = __shfl_xor(h, d, 8), of = __shfl_xor(f, d, 8);
            h = oh < h ? oh : h;
            f = of < f ? of : f;
        }
        h = bcast(h);
        f = bcast(f);
        if (h >= Ep) break;
        // past a silence longer than any interval nothing handed on reaches
        if ((U)h - (U)te > (U(1) << 30)) nc = 0;
        const int64_t shift = E::kRel ? (int64_t)(((uint64_t)h - (uint64_t)h0) << E::kUp) : 0;
        h0 = h;
        te = f < Ep ? f : Ep;
        if constexpr (E::kRel)
            if ((uint64_t)te - (uint64_t)h > E::kSpan) te = (T)((uint64_t)h + E::kSpan);
        const Key te_k = E::key(te, h);
        const bool all = h >= Bp;
        const int32_t cnt0 = cnt;
        int n = 0;  // entries of the previous node's list
        for (int k = 0; k < N; ++k) {
            T v[kR];
            Key xs[kR];
            uint32_t st[kR];  // start bits
            uint64_t ok[kR];
            int nx = 0;
#pragma unroll
            for (int r = 0; r < kR; ++r) {
                v[r] = x[r];
                ok[r] = __ballot(v[r] < te);
                xs[r] = E::key(v[r], h);
            }
            if (left < kCap) {
#pragma unroll
                for (int r = 0; r < kR; ++r) ok[r] &= lanes_below(left - r * kW);
            }
#pragma unroll
            for (int r = 0; r < kR; ++r) nx += __popcll(ok[r]);
            if (lane == k) ep.cur += nx;
            // the next node's events, ahead of this node's work
            if (k + 1 == N) load_heads(ts, ep, hv, fv);
            left = load_events(ts, ep, k + 1 < N ? k + 1 : 0, lane, x);
            const int pb = (k & 1) ^ 1, qb = k & 1;  // previous list, this node's list
            if (k == 0) {
#pragma unroll
                for (int r = 0; r < kR; ++r) st[r] = E::start_bits(v[r]);
            } else if (n == 0 || nx == 0) {
#pragma unroll
                for (int r = 0; r < kR; ++r) {
                    st[r] = 0;
                    ok[r] = 0;
                }
            } else {
                const UKey lo = E::len(rdlane(ep.lo, k - 1)), hi = E::len(rdlane(ep.hi, k - 1));
                auto search = [&](auto chunks) __attribute__((always_inline)) {
                    constexpr int NR = decltype(chunks)::value;
                    Key q[NR];
                    uint32_t p[NR];  // byte offset of the latest entry known to be before q
                    const char *list = reinterpret_cast<const char *>(w.e);
                    const uint32_t base = (uint32_t)pb * (uint32_t)sizeof(w.e[0]);
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        q[r] = (Key)((UKey)xs[r] - lo);
                        p[r] = base;
                    }
                    // halving search of the sentinel and the n entries, one length for all
                    int len = n + 1;
                    while (len > 1) {
                        const int half = len >> 1;
                        const uint32_t hb = (uint32_t)half * 8u;
#pragma unroll
                        for (int r = 0; r < NR; ++r) {
                            const uint32_t m = p[r] + hb;
                            p[r] = *reinterpret_cast<const Key *>(list + m + E::kKeyAt) < q[r] ? m : p[r];
                        }
                        len -= half;
                    }
#pragma unroll
                    for (int r = 0; r < NR; ++r) {
                        // (the entry's start bits only lower the difference, by less than one unit of time)
                        const int64_t y = *reinterpret_cast<const int64_t *>(list + p[r]);
                        ok[r] &= __ballot((UKey)xs[r] - E::key_of(y) <= hi);
                        st[r] = E::start_bits((T)y);
                    }
                };
                // where another of the episode's types is much busier, one chunk holds the
                // events of this one
                if (nx <= kW) search(Chunks<1>());
                else search(Chunks<kR>());
            }
            if (k + 1 < N) {
                // this node's list: what it handed on, then the hits in order
                n = rdlane(nc, k);
#pragma unroll
                for (int j = 0; j < HC; ++j) {
                    const int i = j * kW + lane;
                    if (i < n) w.e[qb][1 + i] = (int64_t)((uint64_t)w.c[k][i] - (uint64_t)shift);
                }
#pragma unroll
                for (int r = 0; r < kR; ++r) {
                    const int o = below(ok[r], n + 1);
                    if (in_mask(ok[r])) w.e[qb][o] = E::make(xs[r], st[r]);
                    n += __popcll(ok[r]);
                }
                lds_order();
                // what later windows can reach
                const UKey lo = E::len(rdlane(ep.lo, k)), hi = E::len(rdlane(ep.hi, k));
                int64_t y[HC];
                int fut = 0, live = 0;
#pragma unroll
                for (int j = 0; j < HC; ++j) {
                    const int i = n - HC * kW + j * kW + lane;
                    y[j] = 0;
                    UKey d = ~UKey(0);  // from the entry to the window's end
                    if (i >= 0) {
                        y[j] = w.e[qb][1 + i];
                        d = (UKey)te_k - E::key_of(y[j]);
                    }
                    fut += __popcll(__ballot(d <= lo));
                    live += __popcll(__ballot(d <= hi));
                }
                const int keep = fut + 1 < live ? fut + 1 : live;
#pragma unroll
                for (int j = 0; j < HC; ++j) {
                    const int o = j * kW + lane - (HC * kW - keep);
                    if (o >= 0) w.c[k][o] = y[j];
                }
                if (lane == k) nc = keep;
                lds_order();
            } else {
                // the greedy of Alg. 1
                const bool plain = !SYNC && all && (!first_out || cnt >= kRecFirst);
#pragma unroll
                for (int r = 0; r < kR; ++r) {
                    if (ok[r] == 0) continue;
                    const T L = E::start(v[r], st[r]);
                    uint64_t m = __ballot(L > tau) & ok[r];
                    if (plain && __popcll(ok[r]) > kRunMin) {
                        // many hits: from a kept one on, all hits are kept up to the first that
                        // starts at or before the hit ahead of it (one step a run)
                        const uint64_t before = ok[r] & ((uint64_t(1) << lane) - 1);
                        const T pv = __shfl(v[r], before ? 63 - __clzll(before) : 0, kW);
                        const uint64_t stop = ok[r] & ~__ballot(L > pv);
                        while (m) {
                            const uint64_t from = ~uint64_t(0) << __builtin_ctzll(m);
                            const uint64_t end = stop & (from << 1);
                            const uint64_t run = ok[r] & from & (end ? (end & -end) - 1 : ~uint64_t(0));
                            cnt += __popcll(run);
                            tau = rdlane(v[r], 63 - __builtin_clzll(run));
                            m = __ballot(L > tau) & ok[r];
                        }
                    }
                    while (m) {
                        tau = rdlane(v[r], __builtin_ctzll(m));
                        if (all || tau >= Bp) {
                            if constexpr (SYNC) {
                                int hit = -1;
#pragma unroll
                                for (int j = 0; j < kRecFirst; ++j)
                                    if (j < rec->c && rec->first[j] == tau) hit = j;
                                if (hit >= 0) {
                                    out.cnt = cnt + 1 + (rec->c - hit - 1);
                                    out.synced = true;
                                    return;
                                }
                            } else if (first_out && cnt < kRecFirst) {
                                if (lane == 0) first_out[cnt * first_stride] = tau;
                            }
                            ++cnt;
                        }
                        m = __ballot(L > tau) & ok[r];
                    }
                }
            }
        }
        if (cnt != cnt0) out.last = tau;
        if constexpr (SYNC) {
            // no completion of either run up to here, and no partial
            // occurrence from before Bp left: the states agree
            if (cnt == 0 && te >= rec->sync_t && (rec->c == 0 || rec->first[0] >= te)) {
                out.cnt = rec->c;
                out.synced = true;
                return;
            }
        }
    }
    out.cnt = cnt;
}

template <typename T>
__device__ __forceinline__ int64_t slot_of(const CountArgs<T> &a, int64_t s) {
    return a.perm ? (int64_t)bcast(a.perm[a.begin + s]) : a.begin + s;
}

// Segment p's first and end time.
template <typename T>
__device__ __forceinline__ void seg_bounds(const CountArgs<T> &a, const WaveEp<T> &ep, int p, T &Bp, T &Ep) {
    const int64_t b0 = (int64_t)p * ep.S;
    const int64_t b1 = b0 + ep.S < a.B ? b0 + ep.S : a.B;
    Bp = bcast(p == 0 ? TsLimits<T>::lo() : a.tile_t0[b0]);
    Ep = bcast(p == ep.P - 1 ? TsLimits<T>::hi() : a.tile_t0[b1]);
}

// Candidate s of unit a over segment p: the whole count (P = 1) or the
// segment's speculative record.
template <typename T, int HC>
__device__ __forceinline__ void wave_item(const CountArgs<T> &a, int64_t s, int p, WaveLds<HC> &w, int lane) {
    constexpr T kMin = TsLimits<T>::lo();
    const int64_t slot = slot_of(a, s);
    WaveEp<T> ep = load_episode(a, slot, lane);
    if (p >= ep.P) return;
    const bool whole = ep.P == 1;
    T Bp, Ep;
    seg_bounds(a, ep, p, Bp, Ep);
    T e0 = kMin;
    if (p > 0) {
        e0 = (T)(Bp - ep.H - 1);
        seek((Times<T>)a.ts_by_type, ep, e0, lane);
    }
    WaveOut<T> out;
    out.last = kMin;
    const int64_t ro = (int64_t)p * a.G + s;
    T *first = !whole ? a.rec_first + (int64_t)p * kRecFirst * a.G + s : nullptr;
    wave_run<T, false>((Times<T>)a.ts_by_type, w, ep, e0, Bp, Ep, lane, first, a.G, nullptr, out);
    if (lane == 0) {
        if (whole) {
            const int64_t o = a.orig[slot];
            a.counts[o] = out.cnt;
            if (a.tau) a.tau[o] = out.last;
        } else {
            a.rec_cnt[ro] = out.cnt;
            a.rec_last[ro] = out.last;
        }
    }
    rejoin();
}

// Segment p's completions and last completion given the last completion tau
// before it (see rerun_segment in epi_tiled.hip).
template <typename T, int HC>
__device__ __forceinline__ int32_t wave_fix_segment(const CountArgs<T> &a, int64_t s, int p, T &tau, WaveLds<HC> &w,
                                                    int lane, const WaveEp<T> &ep0) {
    T Bp, Ep;
    seg_bounds(a, ep0, p, Bp, Ep);
    const int64_t ro = (int64_t)p * a.G + s;
    const int32_t c = bcast(a.rec_cnt[ro]);
    const T last = bcast(a.rec_last[ro]);
    if (p == 0 || tau < (T)(Bp - ep0.H)) {
        if (c > 0) tau = last;
        return c;
    }
    WaveRec<T> rec;
    rec.c = c;
    rec.sync_t = (T)(Bp + ep0.H);
#pragma unroll
    for (int j = 0; j < kRecFirst; ++j)
        rec.first[j] = j < c ? bcast(a.rec_first[((int64_t)p * kRecFirst + j) * a.G + s]) : TsLimits<T>::hi();
    WaveEp<T> ep = ep0;
    seek((Times<T>)a.ts_by_type, ep, tau, lane);
    WaveOut<T> out;
    out.last = tau;
    wave_run<T, true>((Times<T>)a.ts_by_type, w, ep, tau, TsLimits<T>::lo(), Ep, lane, nullptr, 0, &rec, out);
    if (out.synced) {
        if (c > 0) tau = last;
    } else {
        tau = out.last;
    }
    return out.cnt;
}

// Pre-pass of candidate s, segment p >= 1: its true completions if the earlier
// records' last completion is the true one.
template <typename T, int HC>
__device__ __forceinline__ void wave_pre(const CountArgs<T> &a, int64_t s, int p, WaveLds<HC> &w, int lane) {
    const WaveEp<T> ep = load_episode(a, slot_of(a, s), lane);
    if (p >= ep.P) return;
    T tau = TsLimits<T>::lo();
    for (int q = p - 1; q >= 0; --q) {
        if (bcast(a.rec_cnt[(int64_t)q * a.G + s]) > 0) {
            tau = bcast(a.rec_last[(int64_t)q * a.G + s]);
            break;
        }
    }
    const T tau0 = tau;
    const int32_t c = wave_fix_segment(a, s, p, tau, w, lane, ep);
    if (lane == 0) {
        const int64_t o = (int64_t)p * a.G + s;
        a.pre_tau[o] = tau0;
        a.pre_cnt[o] = c;
        a.pre_last[o] = tau;
    }
    rejoin();
}

// The count of candidate s from its segments: the pre-pass's results where the
// last completion they assumed is the true one (all lanes test 64 segments at
// once), a re-run elsewhere.
template <typename T, int HC>
__device__ __forceinline__ void wave_sum(const CountArgs<T> &a, int64_t s, WaveLds<HC> &w, int lane) {
    const int64_t slot = slot_of(a, s);
    const WaveEp<T> ep = load_episode(a, slot, lane);
    if (ep.P == 1) return;  // counted whole
    T tau = TsLimits<T>::lo();
    int32_t total = bcast(a.rec_cnt[s]);
    if (total > 0) tau = bcast(a.rec_last[s]);
    int p = 1;
    while (p < ep.P) {
        const int i = p + lane;
        const int64_t o = (int64_t)i * a.G + s;
        const bool in = i < ep.P;
        int32_t c = 0;
        T assumed = 0, end = 0;
        if (in) {
            c = a.pre_cnt[o];
            assumed = a.pre_tau[o];
            end = a.pre_last[o];
        }
        // the true last completion before segment i, if all before it held
        const T prev = __shfl_up(end, 1, kW);
        const uint64_t bad = __ballot(in && assumed != (lane == 0 ? tau : prev));
        const int good = bad ? __builtin_ctzll(bad) : (ep.P - p < kW ? ep.P - p : kW);
        int32_t v = lane < good ? c : 0;
        for (int d = 1; d < kW; d <<= 1) v += __shfl_xor(v, d, kW);
        total += bcast(v);
        if (good > 0) tau = bcast((T)__shfl(end, good - 1, kW));
        p += good;
        if (bad) {
            total += wave_fix_segment(a, s, p, tau, w, lane, ep);
            ++p;
        }
    }
    if (lane == 0) {
        const int64_t o = a.orig[slot];
        a.counts[o] = total;
        if (a.tau) a.tau[o] = tau;
    }
    rejoin();
}

template <typename T, int HC>
__global__ __launch_bounds__(kW) void k_wave_count(CountArgs<T> a) {
    __shared__ WaveLds<HC> w;
    wave_item<T>(a, blockIdx.x, blockIdx.y, w, threadIdx.x);
}

template <typename T, int HC>
__global__ __launch_bounds__(kW) void k_wave_pre(CountArgs<T> a) {
    __shared__ WaveLds<HC> w;
    wave_pre<T>(a, blockIdx.x, blockIdx.y + 1, w, threadIdx.x);
}

template <typename T, int HC>
__global__ __launch_bounds__(kW) void k_wave_sum(CountArgs<T> a) {
    __shared__ WaveLds<HC> w;
    wave_sum<T>(a, blockIdx.x, w, threadIdx.x);
}

// Appended events (see k_count_append in epi_tiled.hip): the run resumes right
// after max(tau, B - H - 1); every completion it finds is at or after B.
template <typename T, int HC>
__global__ __launch_bounds__(kW) void k_wave_append(CountArgs<T> a, T B) {
    __shared__ WaveLds<HC> w;
    const int lane = threadIdx.x;
    const int64_t s = blockIdx.x;
    const int64_t slot = slot_of(a, s);
    WaveEp<T> ep = load_episode(a, slot, lane);
    const int64_t o = bcast(a.orig[slot]);
    const T tau = bcast(a.tau[o]);
    const T from = tau > (T)(B - ep.H - 1) ? tau : (T)(B - ep.H - 1);
    seek((Times<T>)a.ts_by_type, ep, from, lane);
    WaveOut<T> out;
    out.last = tau;
    wave_run<T, false>((Times<T>)a.ts_by_type, w, ep, from, TsLimits<T>::lo(), TsLimits<T>::hi(), lane, nullptr, 0, nullptr, out);
    if (lane == 0) {
        a.counts[o] += out.cnt;
        a.tau[o] = out.last;
    }
}

// Batched form.  A work item is (unit, block of 64 slots, segment); a wave
// takes one slot of it at a time from the queue.  Where episodes have fewer
// segments than their unit, most slots of an item are empty (12,500 episodes
// over skewed rates: 137,000 slots, 26,000 of them at work), and the queue's
// one counter takes about 5 ns a slot: the slots at work are listed first, in
// the items' order, and the queue runs over the list (with half as many
// segments again, which the list makes cheap: 5.4 ms -> 4.6 ms; 438 episodes
// of 1-2 nodes over skewed rates: 2.3 ms -> 0.52).  Light slots come several at
// a turn (WaveSlots::take).
// masks[i]: item i's slots at work.
template <typename T>
__global__ __launch_bounds__(kW) void k_wave_live(const CountArgs<T> *__restrict__ units,
                                                  const WorkItem *__restrict__ items,
                                                  unsigned long long *__restrict__ masks) {
    const WorkItem it = items[blockIdx.x];
    const CountArgs<T> &a = units[it.unit];
    const int64_t s = it.blk * kW + threadIdx.x;
    bool live = s < a.G;
    if (live && it.p > 0) {
        const int64_t slot = a.perm ? (int64_t)a.perm[a.begin + s] : a.begin + s;
        const int N = a.cN[slot];
        int64_t c = 0;
        for (int k = 0; k < N; ++k) {
            const int32_t ty = a.ctypes[(int64_t)k * a.m + slot];
            c += a.type_off[ty + 1] - a.type_off[ty];
        }
        int32_t P;
        int64_t S;
        own_segments(a, c, P, S);
        live = it.p < P;
    }
    const uint64_t m = __ballot(live);
    if (threadIdx.x == 0) masks[blockIdx.x] = m;
}

// off[i]: slots at work before item i (one workgroup); off[n]: all.
constexpr int kOffBlock = 1024;
__global__ __launch_bounds__(kOffBlock) void k_wave_offsets(const unsigned long long *__restrict__ masks, int64_t n,
                                                            int64_t *__restrict__ off) {
    __shared__ int64_t sum[2][kOffBlock / kW];
    const int lane = threadIdx.x % kW, w = threadIdx.x / kW;
    int64_t carry = 0;
    int b = 0;
    for (int64_t i0 = 0; i0 < n; i0 += kOffBlock, b ^= 1) {
        const int64_t i = i0 + threadIdx.x;
        const int own = i < n ? __popcll(masks[i]) : 0;
        int x = own;
        for (int d = 1; d < kW; d <<= 1) {
            const int y = __shfl_up(x, d, kW);
            if (lane >= d) x += y;
        }
        if (lane == kW - 1) sum[b][w] = x;
        __syncthreads();
        int64_t at = carry + x - own;
        for (int k = 0; k < kOffBlock / kW; ++k) {
            if (k < w) at += sum[b][k];
            carry += sum[b][k];
        }
        if (i < n) off[i] = at;
    }
    if (threadIdx.x == 0) off[n] = carry;
}

__global__ __launch_bounds__(kW) void k_wave_list(const unsigned long long *__restrict__ masks,
                                                  const int64_t *__restrict__ off, int64_t cap,
                                                  int64_t *__restrict__ list) {
    const uint64_t m = masks[blockIdx.x];
    const int64_t o = off[blockIdx.x] + below(m, 0);
    if (((m >> threadIdx.x) & 1) && o < cap) list[o] = (int64_t)blockIdx.x * kW + threadIdx.x;
}

// The slots of a batched launch: all of the items', or those listed.
struct WaveSlots {
    const WorkItem *items;
    int64_t n_items;
    const int64_t *list;   // null: all
    const int64_t *total;  // listed slots
    int64_t cap;
    int take;              // slots a wave takes from the queue at a time
    __device__ __forceinline__ int64_t count() const {
        if (!list) return n_items * kW;
        const int64_t t = bcast(*total);
        return t < cap ? t : cap;
    }
    __device__ __forceinline__ int64_t at(int64_t q) const { return list ? bcast(list[q]) : q; }
};

template <typename T, int HC>
__global__ __launch_bounds__(kW) void k_wave_persistent(const CountArgs<T> *__restrict__ units, WaveSlots slots,
                                                        unsigned long long *__restrict__ queue) {
    __shared__ WaveLds<HC> w;
    const int lane = threadIdx.x;
    const int64_t n = slots.count();
    while (true) {
        rejoin();
        int64_t q0 = 0;
        if (lane == 0) q0 = (int64_t)atomicAdd(queue, (unsigned long long)slots.take);
        rejoin();
        q0 = bcast(q0);
        // unsigned: any counter value beyond the slots ends the loop
        if ((uint64_t)q0 >= (uint64_t)n) break;
        for (int64_t i = q0; i < n && i < q0 + slots.take; ++i) {
            const int64_t q = slots.at(i);
            const WorkItem it = slots.items[q / kW];
            const CountArgs<T> &a = units[it.unit];
            const int64_t s = it.blk * kW + (q % kW);
            if (s < a.G) wave_item<T>(a, s, it.p, w, lane);
        }
    }
}

template <typename T, int HC>
__global__ __launch_bounds__(kW) void k_wave_pre_all(const CountArgs<T> *__restrict__ units, WaveSlots slots) {
    __shared__ WaveLds<HC> w;
    const int64_t n = slots.count();
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int64_t q = slots.at(i);
        const WorkItem it = slots.items[q / kW];
        const CountArgs<T> &a = units[it.unit];
        const int64_t s = it.blk * kW + (q % kW);
        if (s < a.G && it.p > 0) wave_pre<T>(a, s, it.p, w, threadIdx.x);
    }
}

template <typename T, int HC>
__global__ __launch_bounds__(kW) void k_wave_sum_all(const CountArgs<T> *__restrict__ units, WaveSlots slots) {
    __shared__ WaveLds<HC> w;
    const int64_t n = slots.count();
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int64_t q = slots.at(i);
        const WorkItem it = slots.items[q / kW];
        const CountArgs<T> &a = units[it.unit];
        const int64_t s = it.blk * kW + (q % kW);
        if (s < a.G && it.p == 0 && a.P > 1) wave_sum<T>(a, s, w, threadIdx.x);
    }
}

constexpr int64_t kMostWaves = (int64_t(1) << 32) / kW - 1;  // of a grid's first dimension

unsigned grid_of(int64_t n) { return (unsigned)std::min<int64_t>(std::max<int64_t>(n, 1), int64_t(1) << 16); }

}  // namespace

int wave_waves_per_cu(int hand) {
    int per = 0;
    const void *fn = hand == 1 ? (const void *)k_wave_persistent<int64_t, 1> : (const void *)k_wave_persistent<int64_t, 2>;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kW, 0) != hipSuccess || per < 1) {
        (void)hipGetLastError();
        per = 8;
    }
    return per;
}

namespace {

template <typename T, int HC>
hipError_t launch_hand(const CountArgs<T> &a, hipStream_t st) {
    k_wave_count<T, HC><<<dim3((unsigned)a.G, (unsigned)a.P), kW, 0, st>>>(a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.P == 1) return e;
    k_wave_pre<T, HC><<<dim3((unsigned)a.G, (unsigned)(a.P - 1)), kW, 0, st>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_wave_sum<T, HC><<<(unsigned)a.G, kW, 0, st>>>(a);
    return hipGetLastError();
}

template <typename T, int HC>
hipError_t persistent_hand(unsigned grid, hipStream_t st, const CountArgs<T> *units, const WaveSlots &slots,
                           unsigned long long *queue, bool segmented, unsigned all) {
    k_wave_persistent<T, HC><<<grid, kW, 0, st>>>(units, slots, queue);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !segmented) return e;
    k_wave_pre_all<T, HC><<<all, kW, 0, st>>>(units, slots);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_wave_sum_all<T, HC><<<all, kW, 0, st>>>(units, slots);
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t wave_launch(const CountArgs<T> &a, int hand, hipStream_t st) {
    if (a.G <= 0) return hipSuccess;
    if (a.P < 1 || a.P > 65535 || !a.cN || !a.orig || a.G > kMostWaves) return hipErrorInvalidValue;
    return hand == 1 ? launch_hand<T, 1>(a, st) : launch_hand<T, 2>(a, st);
}

template <typename T>
hipError_t wave_launch_append(const CountArgs<T> &a, int hand, T B, hipStream_t st) {
    if (a.G <= 0) return hipSuccess;
    if (!a.cN || !a.orig || !a.tau || a.G > kMostWaves) return hipErrorInvalidValue;
    if (hand == 1) k_wave_append<T, 1><<<(unsigned)a.G, kW, 0, st>>>(a, B);
    else k_wave_append<T, 2><<<(unsigned)a.G, kW, 0, st>>>(a, B);
    return hipGetLastError();
}

size_t wave_list_bytes(int64_t n_items, int64_t cap) {
    return sizeof(int64_t) * (size_t)(2 * n_items + 1 + cap);
}

template <typename T>
hipError_t wave_launch_persistent(unsigned grid, int hand, hipStream_t st, const CountArgs<T> *units,
                                  const WorkItem *items, int64_t n_items, unsigned long long *queue, bool segmented,
                                  void *list, int64_t cap, int take) {
    WaveSlots slots{items, n_items, nullptr, nullptr, cap, take};
    if (list) {
        if (n_items > kMostWaves) return hipErrorInvalidValue;
        int64_t *off = static_cast<int64_t *>(list), *out = off + n_items + 1;
        auto *masks = reinterpret_cast<unsigned long long *>(out + cap);
        k_wave_live<T><<<(unsigned)n_items, kW, 0, st>>>(units, items, masks);
        k_wave_offsets<<<1, kOffBlock, 0, st>>>(masks, n_items, off);
        k_wave_list<<<(unsigned)n_items, kW, 0, st>>>(masks, off, cap, out);
        slots.list = out;
        slots.total = off + n_items;
    }
    const unsigned all = grid_of(list ? cap : n_items * kW);
    return hand == 1 ? persistent_hand<T, 1>(grid, st, units, slots, queue, segmented, all)
                     : persistent_hand<T, 2>(grid, st, units, slots, queue, segmented, all);
}

template hipError_t wave_launch<int32_t>(const CountArgs<int32_t> &, int, hipStream_t);
template hipError_t wave_launch<int64_t>(const CountArgs<int64_t> &, int, hipStream_t);
template hipError_t wave_launch_append<int32_t>(const CountArgs<int32_t> &, int, int32_t, hipStream_t);
template hipError_t wave_launch_append<int64_t>(const CountArgs<int64_t> &, int, int64_t, hipStream_t);
template hipError_t wave_launch_persistent<int32_t>(unsigned, int, hipStream_t, const CountArgs<int32_t> *,
                                                    const WorkItem *, int64_t, unsigned long long *, bool, void *, int64_t, int);
template hipError_t wave_launch_persistent<int64_t>(unsigned, int, hipStream_t, const CountArgs<int64_t> *,
                                                    const WorkItem *, int64_t, unsigned long long *, bool, void *, int64_t, int);

}  // namespace epi
