// Per-type index of an event stream (the pre-processing step of Sec. IV-A):
// the events of each type, in time order, stored contiguously.
//
//   0. k_ingest:  copies and checks the events, and takes what the tile size is
//                 chosen by: the longest tile of each size the stream may pick.
//   1. k_hist:    one workgroup per tile; LDS histogram over the K types; writes
//                 cnt[tile][type] (tile-major: coalesced).
//   2. column scans: exclusive prefix sums down the tiles of each type, in three
//                 passes (chunks of tiles, the chunks and the types, the tiles);
//                 base[tile][type] is then the global output position of the
//                 tile's first event of that type, and a type's first tile's is
//                 the type's offset.
//   3. k_scatter: one workgroup per tile orders the tile's events by type in LDS,
//                 stably: every wave takes a stretch of the tile, counts its
//                 types, and ranks 64 events at a time among the equal types of
//                 the wave by ballots over the type's bits.  The ordered tile is
//                 the tile-major copy (each tile's events grouped by type, with
//                 per-tile uint16 offsets, so that a workgroup can stage a time
//                 window of every type list with one contiguous copy) and, run by
//                 run, the per-type index: times, and the stream position of
//                 every entry.
//
// What bounds it: memory.  20 bytes an event read and 20 written (int64 times),
// the per-type index in runs of a tile's events of a type; neighbouring tiles go
// to one XCD, whose L2 joins their runs to whole lines.  One wave a tile with 64
// broadcasts for each rank took 451 us for 9M events of 128 types; now 97 us (3.7 TB/s).
#include <algorithm>
#include <cstring>
#include <vector>

#include "epi_count.h"

namespace epi {

namespace {

constexpr int kWave = 64;
constexpr int kIdxBlock = 256;               // threads of a tile's workgroup
constexpr int kIdxWaves = kIdxBlock / kWave;
constexpr int kXcds = 8;

// Tile of a workgroup: workgroups go to the XCDs in turn, so each XCD takes a
// stretch of neighbouring tiles.
__device__ __forceinline__ int64_t tile_of(int64_t blk, int64_t B) {
    const int64_t per = (B + kXcds - 1) / kXcds;
    return (blk % kXcds) * per + blk / kXcds;  // (>= B: none)
}
inline unsigned tile_grid(int64_t B) { return (unsigned)((B + kXcds - 1) / kXcds * kXcds); }

__global__ __launch_bounds__(kIdxBlock) void k_hist(const int32_t *__restrict__ types, int64_t n, int32_t K,
                                                    int32_t TT, int64_t B, int32_t *__restrict__ cnt) {
    extern __shared__ int32_t h[];
    const int64_t b = tile_of(blockIdx.x, B);
    if (b >= B) return;
    for (int k = threadIdx.x; k < K; k += kIdxBlock) h[k] = 0;
    __syncthreads();
    const int64_t beg = b * TT;
    const int64_t end = beg + TT < n ? beg + TT : n;
    for (int64_t i = beg + threadIdx.x; i < end; i += kIdxBlock) atomicAdd(&h[types[i]], 1);
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += kIdxBlock) cnt[b * K + k] = h[k];
}

// Column scans of cnt[B][K]: chunks of kColTiles tiles.
constexpr int kColTiles = 32;

// sums[c][k] = the chunk's events of type k
__global__ __launch_bounds__(kIdxBlock) void k_col_sum(const int32_t *__restrict__ cnt, int64_t B, int32_t K,
                                                       int32_t *__restrict__ sums) {
    const int k = blockIdx.y * kIdxBlock + threadIdx.x;
    if (k >= K) return;
    const int64_t b0 = (int64_t)blockIdx.x * kColTiles;
    const int64_t b1 = b0 + kColTiles < B ? b0 + kColTiles : B;
    int32_t acc = 0;
#pragma unroll 8
    for (int64_t b = b0; b < b1; ++b) acc += cnt[b * K + k];
    sums[(int64_t)blockIdx.x * K + k] = acc;
}

// tot[k] = the type's events; sums become the exclusive sums down the chunks.
// One wave a type: 64 chunks at a time.
__global__ __launch_bounds__(kWave) void k_col_chunks(int32_t *__restrict__ sums, int64_t nc, int32_t K,
                                                      int32_t *__restrict__ tot) {
    const int k = blockIdx.x, lane = threadIdx.x;
    int32_t carry = 0;
    for (int64_t c0 = 0; c0 < nc; c0 += kWave) {
        const int64_t c = c0 + lane;
        const int32_t v = c < nc ? sums[c * K + k] : 0;
        int32_t x = v;
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t y = __shfl_up(x, d, kWave);
            if (lane >= d) x += y;
        }
        if (c < nc) sums[c * K + k] = carry + x - v;
        carry += __shfl(x, kWave - 1, kWave);
    }
    if (lane == 0) tot[k] = carry;
}

// off[k] = exclusive sum of tot over the types (one workgroup), off[K] = n.
__global__ __launch_bounds__(kIdxBlock) void k_type_off(const int32_t *__restrict__ tot, int32_t K,
                                                        int32_t *__restrict__ off) {
    __shared__ int32_t wsum[kIdxWaves];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    int32_t carry = 0;
    for (int k0 = 0; k0 < K; k0 += kIdxBlock) {
        const int k = k0 + threadIdx.x;
        const int32_t v = k < K ? tot[k] : 0;
        int32_t x = v;
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t y = __shfl_up(x, d, kWave);
            if (lane >= d) x += y;
        }
        if (lane == kWave - 1) wsum[w] = x;
        __syncthreads();
        int32_t before = 0, all = 0;
        for (int i = 0; i < kIdxWaves; ++i) {
            if (i < w) before += wsum[i];
            all += wsum[i];
        }
        __syncthreads();
        if (k < K) off[k] = carry + before + x - v;
        carry += all;
    }
    if (threadIdx.x == 0) off[K] = carry;
}

// base[b][k] (in place of cnt): the output position of tile b's first event of
// type k.
__global__ __launch_bounds__(kIdxBlock) void k_col_apply(int32_t *__restrict__ cnt, int64_t B, int32_t K,
                                                         const int32_t *__restrict__ sums,
                                                         const int32_t *__restrict__ off) {
    const int k = blockIdx.y * kIdxBlock + threadIdx.x;
    if (k >= K) return;
    const int64_t b0 = (int64_t)blockIdx.x * kColTiles;
    const int64_t b1 = b0 + kColTiles < B ? b0 + kColTiles : B;
    int32_t run = off[k] + sums[(int64_t)blockIdx.x * K + k];
#pragma unroll 8
    for (int64_t b = b0; b < b1; ++b) {
        const int32_t v = cnt[b * K + k];
        cnt[b * K + k] = run;
        run += v;
    }
}

// LDS of k_scatter: the ordered tile (times, positions, types), per-wave running
// positions of every type, each type's first position.
template <typename T>
size_t scatter_lds(int32_t K, int32_t TT) {
    return (size_t)TT * (sizeof(T) + 2 * sizeof(uint16_t)) + sizeof(uint16_t) * (size_t)(kIdxWaves + 1) * K;
}

// bits: of the largest type
template <typename T>
__global__ __launch_bounds__(kIdxBlock) void k_scatter(const int32_t *__restrict__ types, const T *__restrict__ times,
                                                       int64_t n, int32_t K, int bits, int64_t B,
                                                       const int32_t *__restrict__ base, T *__restrict__ out,
                                                       int32_t *__restrict__ pos_out, T *__restrict__ tiled,
                                                       uint16_t *__restrict__ loff, T *__restrict__ tile_t0,
                                                       int32_t TT) {
    extern __shared__ __align__(16) unsigned char smem[];
    T *st = reinterpret_cast<T *>(smem);
    uint16_t *sp = reinterpret_cast<uint16_t *>(st + TT), *sy = sp + TT;
    uint16_t *run = sy + TT;             // [wave][K]
    uint16_t *start = run + kIdxWaves * K;  // [K]
    __shared__ int32_t wsum[kIdxWaves];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int64_t b = tile_of(blockIdx.x, B);
    if (b >= B) return;
    const int64_t beg = b * TT;
    const int m = (int)(beg + TT < n ? TT : n - beg);  // events of the tile
    for (int k = threadIdx.x; k < kIdxWaves * K; k += kIdxBlock) run[k] = 0;
    __syncthreads();
    // each wave's stretch of the tile (TT is a multiple of the workgroup's lanes)
    const int per = TT / kIdxWaves, r0 = w * per, r1 = r0 + per < m ? r0 + per : m;
    uint16_t *mine = run + w * K;
    // equal types of a wave's 64 events: the lanes that agree in every bit
    auto peers = [&](int32_t ty, uint64_t in) {
        uint64_t p = in;
        for (int q = 0; q < bits; ++q) {
            const bool one = (ty >> q) & 1;
            const uint64_t v = __ballot(one);
            p &= one ? v : ~v;
        }
        return p;
    };
    for (int r = r0; r < r1; r += kWave) {
        const bool in = r + lane < r1;
        const int32_t ty = in ? types[beg + r + lane] : 0;
        const uint64_t p = peers(ty, __ballot(in));
        if (in && (p >> lane) == 1) mine[ty] += (uint16_t)__popcll(p);  // the last of them
    }
    __syncthreads();
    // tile-local offsets: exclusive sums over the types, each wave's after the
    // ones before it
    int32_t carry = 0;
    for (int k0 = 0; k0 < K; k0 += kIdxBlock) {
        const int k = k0 + threadIdx.x;
        int32_t c[kIdxWaves], v = 0;
        for (int i = 0; i < kIdxWaves; ++i) {
            c[i] = k < K ? run[i * K + k] : 0;
            v += c[i];
        }
        int32_t x = v;
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t y = __shfl_up(x, d, kWave);
            if (lane >= d) x += y;
        }
        if (lane == kWave - 1) wsum[w] = x;
        __syncthreads();
        int32_t o = carry + x - v, all = 0;
        for (int i = 0; i < kIdxWaves; ++i) {
            if (i < w) o += wsum[i];
            all += wsum[i];
        }
        __syncthreads();
        if (k < K) {
            start[k] = (uint16_t)o;
            loff[b * (K + 1) + k] = (uint16_t)o;
            for (int i = 0; i < kIdxWaves; ++i) {
                run[i * K + k] = (uint16_t)o;
                o += c[i];
            }
        }
        carry += all;
    }
    if (threadIdx.x == 0) {
        loff[b * (K + 1) + K] = (uint16_t)m;
        tile_t0[b] = times[beg];
        if (b == B - 1) tile_t0[B] = TsLimits<T>::hi();
    }
    __syncthreads();
    for (int r = r0; r < r1; r += kWave) {
        const int i = r + lane;
        const bool in = i < r1;
        const int32_t ty = in ? types[beg + i] : 0;
        const T t = in ? times[beg + i] : T(0);
        const uint64_t p = peers(ty, __ballot(in));
        int o = 0;
        if (in) o = mine[ty] + __popcll(p & ((uint64_t(1) << lane) - 1));
        __builtin_amdgcn_wave_barrier();  // (every lane has read before the last of its peers writes)
        if (in) {
            if ((p >> lane) == 1) mine[ty] = (uint16_t)(o + 1);
            st[o] = t;
            sp[o] = (uint16_t)i;
            sy[o] = (uint16_t)ty;
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int q = threadIdx.x; q < m; q += kIdxBlock) {
        const int ty = sy[q];
        const T t = st[q];
        const int64_t d = (int64_t)base[b * K + ty] + (q - (int)start[ty]);
        tiled[beg + q] = t;
        out[d] = t;
        pos_out[d] = (int32_t)(beg + sp[q]);
    }
}

// out[h] = min over events i with an event i + kWaveGap[h] of the same type of
// the time between them (out holds the type's maximum before).
constexpr int kGapBlock = 256, kGapItems = 16;
template <typename T>
__global__ __launch_bounds__(kGapBlock) void k_gap(const T *__restrict__ ts, int64_t n,
                                                   const int32_t *__restrict__ off, int32_t K,
                                                   unsigned long long *__restrict__ out) {
    const int64_t b0 = (int64_t)blockIdx.x * kGapBlock * kGapItems;
    // type of the block's first event: the last with off <= b0
    int lo = 0, hi = K - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (off[mid] <= b0) lo = mid; else hi = mid - 1;
    }
    int ty = lo;
    unsigned long long best[kWaveHands];
    for (int h = 0; h < kWaveHands; ++h) best[h] = INT64_MAX;
    for (int q = 0; q < kGapItems; ++q) {
        const int64_t i = b0 + q * kGapBlock + threadIdx.x;
        if (i + kWaveGap[0] >= n) break;
        while (off[ty + 1] <= i) ++ty;
#pragma unroll
        for (int h = 0; h < kWaveHands; ++h) {
            if (i + kWaveGap[h] < off[ty + 1]) {
                const unsigned long long d = (unsigned long long)ts[i + kWaveGap[h]] - (unsigned long long)ts[i];
                best[h] = d < best[h] ? d : best[h];
            }
        }
    }
    // one atomic a block, and only where it lowers the minimum (a stale read
    // only costs an atomic): thousands on one address would serialise
    __shared__ unsigned long long part[kWaveHands][kGapBlock / kWave];
#pragma unroll
    for (int h = 0; h < kWaveHands; ++h) {
        for (int d = 1; d < kWave; d <<= 1) {
            const unsigned long long o = __shfl_xor(best[h], d, kWave);
            best[h] = o < best[h] ? o : best[h];
        }
        if (threadIdx.x % kWave == 0) part[h][threadIdx.x / kWave] = best[h];
    }
    __syncthreads();
    if (threadIdx.x < kWaveHands) {
        unsigned long long b = part[threadIdx.x][0];
        for (int q = 1; q < kGapBlock / kWave; ++q) b = part[threadIdx.x][q] < b ? part[threadIdx.x][q] : b;
        if (b < *(volatile unsigned long long *)(out + threadIdx.x)) atomicMin(out + threadIdx.x, b);
    }
}

__global__ void k_gap_init(unsigned long long *out) { out[threadIdx.x] = INT64_MAX; }

// Tile sizes a stream may pick: kMinTile << q.
constexpr int kTileSizes = 5;
static_assert(kMinTile << (kTileSizes - 1) == kTile, "tile sizes");
// What k_ingest finds out: the longest tile of each size (its first time to the
// next tile's first, or to the last event), a cache line each, and what is wrong
// with the events (IngestBad).
struct IngestInfo {
    static constexpr int kStride = 16;
    unsigned long long span[kTileSizes * kStride];
    unsigned long long cells;  // int64 times: events that begin a stretch of 2^kCellBits units, but the first
    int64_t ends[2];  // the first and the last event's time
    uint32_t bad;
};

// Copies the events (src null: they are in place already), checks them and takes
// the longest tile of each size.
template <typename T>
__global__ __launch_bounds__(kIdxBlock) void k_ingest(const int32_t *__restrict__ src_types,
                                                      const T *__restrict__ src_times, int32_t *__restrict__ types,
                                                      T *__restrict__ times, int64_t n, int32_t K, bool check,
                                                      IngestInfo *__restrict__ info) {
    // a workgroup takes kTile events: few workgroups meet at the maxima
    const int64_t beg = (int64_t)blockIdx.x * kTile, end = beg + kTile < n ? beg + kTile : n;
    const T *tm = src_times ? src_times : times;
    const int32_t *ty = src_types ? src_types : types;
    if (src_types || check) {
        uint32_t bad = 0, cells = 0;
#pragma unroll 4
        for (int64_t i = beg + threadIdx.x; i < end; i += kIdxBlock) {
            const int32_t y = ty[i];
            const T t = tm[i];
            if (src_types) {
                types[i] = y;
                times[i] = t;
            }
            const T next = tm[i + 1 < n ? i + 1 : i];
            if constexpr (sizeof(T) == 8) cells += (next >> kCellBits) != (t >> kCellBits) ? 1 : 0;
            if (check) {
                bad |= (y < 0 || y >= K ? kBadType : 0) |
                       (t == TsLimits<T>::lo() || t == TsLimits<T>::hi() ? kBadTime : 0) |
                       (next < t ? kUnsorted : 0);
            }
        }
        if (bad) atomicOr(&info->bad, bad);
        if constexpr (sizeof(T) == 8) {
            for (int d = 1; d < kWave; d <<= 1) cells += __shfl_xor(cells, d, kWave);
            if (threadIdx.x % kWave == 0 && cells) atomicAdd(&info->cells, (unsigned long long)cells);
        }
    }
    if (threadIdx.x == 0 && beg == 0) info->ends[0] = (int64_t)tm[0];
    if (threadIdx.x == 0 && end == n) info->ends[1] = (int64_t)tm[n - 1];
    // one wave: lane q of 16 the smallest tile q of the stretch, and from their
    // ends the larger tiles
    if (threadIdx.x >= kTile / kMinTile) return;
    const int64_t b0 = beg + (int64_t)threadIdx.x * kMinTile;
#pragma unroll
    for (int q = 0; q < kTileSizes; ++q) {
        unsigned long long d = 0;
        if (b0 < n && (threadIdx.x & ((1u << q) - 1)) == 0) {
            const int64_t b1 = b0 + ((int64_t)kMinTile << q);
            d = (unsigned long long)(int64_t)tm[b1 < n ? b1 : n - 1] - (unsigned long long)(int64_t)tm[b0];
        }
        for (int m = 1; m < kTile / kMinTile; m <<= 1) {
            const unsigned long long o = __shfl_xor(d, m, kTile / kMinTile);
            d = o > d ? o : d;
        }
        unsigned long long *o = &info->span[q * IngestInfo::kStride];
        if (threadIdx.x == 0 && d > *(volatile unsigned long long *)o) atomicMax(o, d);  // (a stale read only costs an atomic)
    }
}

__global__ void k_ingest_init(IngestInfo *info) {
    info->bad = 0;
    info->cells = 0;
    for (int q = 0; q < kTileSizes; ++q) info->span[q * IngestInfo::kStride] = 0;
}

template <typename T>
hipError_t ingest_t(Stream &s, const int32_t *src_types, const T *src_times, bool check, uint32_t *bad,
                    hipStream_t st) {
    hipError_t e;
    DevBuf info;
    if ((e = info.alloc(sizeof(IngestInfo))) != hipSuccess) return e;
    k_ingest_init<<<1, 1, 0, st>>>(info.as<IngestInfo>());
    k_ingest<T><<<(unsigned)((s.n + kTile - 1) / kTile), kIdxBlock, 0, st>>>(
        src_types, src_times, s.types.as<int32_t>(), s.times.as<T>(), s.n, s.K, check, info.as<IngestInfo>());
    if ((e = hipGetLastError()) != hipSuccess) return e;
    IngestInfo h;
    if ((e = hipMemcpyAsync(&h, info.p, sizeof(h), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    *bad = h.bad;
    if (src_types || check) s.cells = sizeof(T) == 8 ? 1 + (int64_t)h.cells : 0;
    s.tmin = h.ends[0];
    s.tmax = h.ends[1];
    for (int q = 0; q < kTileSizes; ++q) {
        const unsigned long long d = h.span[q * IngestInfo::kStride];
        s.tile_span[q] = d > (unsigned long long)INT64_MAX ? INT64_MAX : (int64_t)d;
    }
    return hipSuccess;
}

// Longest tile of T events.
int64_t longest_tile(const Stream &s, int T) {
    int q = 0;
    while ((kMinTile << q) < T) ++q;
    return s.tile_span[q];
}

// Events per tile of a stream (Stream::T).
void pick_tile(Stream &s) {
    const int cap = std::max(kMinTile, std::min(kTile, s.tile_cap));
    s.T = cap;
    if (s.n <= kMinTile) return;
    for (int64_t bound : {(int64_t(1) << 29) - 1, int64_t(1) << 30}) {
        for (int T = cap; T >= kMinTile; T /= 2) {
            if (longest_tile(s, T) < bound) {
                s.T = T;
                return;
            }
        }
    }
}

}  // namespace

hipError_t ingest_stream(Stream &s, const int32_t *src_types, const void *src_times, bool check, uint32_t *bad,
                         hipStream_t st) {
    *bad = 0;
    if (s.n == 0) return hipSuccess;
    if (s.ts_kind == EPI_TS_I64) return ingest_t<int64_t>(s, src_types, (const int64_t *)src_times, check, bad, st);
    return ingest_t<int32_t>(s, src_types, (const int32_t *)src_times, check, bad, st);
}

hipError_t build_type_index(Stream &s, hipStream_t st) {
    hipError_t e;
    const int64_t n = s.n;
    const int32_t K = s.K;
    pick_tile(s);
    const int TT = s.T;
    const int64_t B = n > 0 ? (n + TT - 1) / TT : 0;
    s.B = B;
    s.max_tile_span = n > 0 ? longest_tile(s, TT) : 0;
    for (int64_t &g : s.gap) g = INT64_MAX;
    // (the offsets, and behind them the gaps: one copy brings both to the host)
    const size_t gap_at = (sizeof(int32_t) * ((size_t)K + 1) + 7) & ~(size_t)7;
    if ((e = s.type_off.alloc(gap_at + sizeof(s.gap))) != hipSuccess) return e;
    // (padded: the wave chains load whole windows)
    if ((e = s.ts_by_type.alloc(s.ts_bytes() * ((size_t)n + kWaveChunks * kWave))) != hipSuccess) return e;
    if ((e = s.pos_by_type.alloc(sizeof(int32_t) * (size_t)n)) != hipSuccess) return e;
    if ((e = s.tiled_ts.alloc(s.ts_bytes() * (size_t)B * TT)) != hipSuccess) return e;
    if ((e = s.tile_loff.alloc(sizeof(uint16_t) * (size_t)B * (K + 1))) != hipSuccess) return e;
    if ((e = s.tile_t0.alloc(s.ts_bytes() * (size_t)(B + 1))) != hipSuccess) return e;
    s.h_off.assign(K + 1, 0);
    if (n == 0) {
        if ((e = hipMemsetAsync(s.type_off.p, 0, sizeof(int32_t) * (K + 1), st)) != hipSuccess) return e;
        return hipStreamSynchronize(st);
    }
    const int64_t nc = (B + kColTiles - 1) / kColTiles;
    DevBuf cnt, sums, tot;
    auto *gap = reinterpret_cast<unsigned long long *>(s.type_off.as<char>() + gap_at);
    if ((e = cnt.alloc(sizeof(int32_t) * (size_t)B * K)) != hipSuccess) return e;
    if ((e = sums.alloc(sizeof(int32_t) * (size_t)nc * K)) != hipSuccess) return e;
    if ((e = tot.alloc(sizeof(int32_t) * (size_t)K)) != hipSuccess) return e;
    k_hist<<<tile_grid(B), kIdxBlock, sizeof(int32_t) * (size_t)K, st>>>(s.types.as<int32_t>(), n, K, TT, B,
                                                                       cnt.as<int32_t>());
    const dim3 cols((unsigned)nc, (unsigned)((K + kIdxBlock - 1) / kIdxBlock));
    k_col_sum<<<cols, kIdxBlock, 0, st>>>(cnt.as<int32_t>(), B, K, sums.as<int32_t>());
    k_col_chunks<<<(unsigned)K, kWave, 0, st>>>(sums.as<int32_t>(), nc, K, tot.as<int32_t>());
    k_type_off<<<1, kIdxBlock, 0, st>>>(tot.as<int32_t>(), K, s.type_off.as<int32_t>());
    k_col_apply<<<cols, kIdxBlock, 0, st>>>(cnt.as<int32_t>(), B, K, sums.as<int32_t>(), s.type_off.as<int32_t>());
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int bits = 1;
    while ((K - 1) >> bits) ++bits;
    auto scatter = [&](auto t) -> hipError_t {
        using T = decltype(t);
        const size_t lds = scatter_lds<T>(K, TT);
        hipError_t x;
        if (lds > 64 * 1024 &&
            (x = hipFuncSetAttribute(reinterpret_cast<const void *>(k_scatter<T>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) != hipSuccess)
            return x;
        k_scatter<T><<<tile_grid(B), kIdxBlock, lds, st>>>(
            s.types.as<int32_t>(), s.times.as<T>(), n, K, bits, B, cnt.as<int32_t>(), s.ts_by_type.as<T>(),
            s.pos_by_type.as<int32_t>(), s.tiled_ts.as<T>(), s.tile_loff.as<uint16_t>(), s.tile_t0.as<T>(), TT);
        k_gap_init<<<1, kWaveHands, 0, st>>>(gap);
        if (n > kWaveGap[0])
            k_gap<T><<<(unsigned)((n + kGapBlock * kGapItems - 1) / (kGapBlock * kGapItems)), kGapBlock, 0, st>>>(
                s.ts_by_type.as<T>(), n, s.type_off.as<int32_t>(), K, gap);
        return hipGetLastError();
    };
    if ((e = s.ts_kind == EPI_TS_I64 ? scatter(int64_t()) : scatter(int32_t())) != hipSuccess) return e;
    std::vector<char> host(gap_at + sizeof(s.gap));
    if ((e = hipMemcpyAsync(host.data(), s.type_off.p, host.size(), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    // the temporaries are freed when this returns: wait for the kernels first
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    std::memcpy(s.h_off.data(), host.data(), sizeof(int32_t) * ((size_t)K + 1));
    std::memcpy(s.gap, host.data() + gap_at, sizeof(s.gap));
    return hipSuccess;
}

}  // namespace epi
