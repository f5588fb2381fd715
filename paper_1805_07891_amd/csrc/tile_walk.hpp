// Walks over a wave's tiles and remainders for a compile-time worker count
// (fused_step.hip, fused_stream.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

#include "device.hpp"
#include "kernels.hpp"

namespace phub {

namespace {

// ------------------------------------------------------------ full tiles

// The streams of one full tile: uniform base pointers of the NW gradients
// and of the S state arrays, and the lane's byte offset of its first float4
// from them.  Lane l takes the float4s at tile float4 index l, l + 64,
// l + 128 and l + 192 (kVecPerLane pieces of 1 KB per wave), so every
// access is a uniform base in SGPRs + 32-bit lane offset + immediate.
template <int NW, int S>
struct TileStreams {
    const float* g[NW];
    float* st[S];
    uint32_t off;
    uint32_t vhi;  // float4 index folded into the gradient (and output) bases
};

template <int NW, int S>
__device__ __forceinline__ void tile_bases(TileStreams<NW, S>& s, const DevTile& d,
                                           float* const* state) {
    const uint32_t vlo = d.vec & kVecLowMask;
#pragma unroll
    for (int i = 0; i < S; ++i) s.st[i] = state[i] + d.arena_offset - size_t(vlo) * 4;
    s.off = (vlo + (threadIdx.x & 63u)) * 16u;
}

// Streams of a tile from its key's pointer row in memory (scalar loads).
template <int NW, int S>
__device__ __forceinline__ void tile_streams(TileStreams<NW, S>& s, const DevTile& d,
                                             const float* const* row, float* const* state) {
    const uint32_t vhi = d.vec & ~kVecLowMask;
#pragma unroll
    for (int w = 0; w < NW; ++w) s.g[w] = row[w] + size_t(vhi) * 4;
    s.vhi = vhi;
    tile_bases<NW, S>(s, d, state);
}

// A key's pointer row fetched with one vector load, lane w holding worker
// w's pointer (lanes past the row repeat its last entry).  Held this way
// the next tile's row costs two VGPRs instead of 2 * NW SGPRs, which
// matters while the current tile's pointers still occupy SGPRs.
template <int NW>
__device__ __forceinline__ uint64_t load_row(const float* const* row) {
    const uint32_t l = threadIdx.x & 63u;
    const uint32_t i = l < uint32_t(NW) ? l : uint32_t(NW - 1);
    return ((const PHUB_GLOBAL uint64_t*)row)[i];
}

__device__ __forceinline__ const float* lane_pointer(uint64_t row, int w) {
    const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(row)), w));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(row >> 32)), w));
    return reinterpret_cast<const float*>((uint64_t(hi) << 32) | lo);
}

// Streams of a tile from a pointer row held one per lane.
template <int NW, int S>
__device__ __forceinline__ void tile_streams(TileStreams<NW, S>& s, const DevTile& d,
                                             uint64_t row, float* const* state) {
    const uint32_t vhi = d.vec & ~kVecLowMask;
#pragma unroll
    for (int w = 0; w < NW; ++w) s.g[w] = lane_pointer(row, w) + size_t(vhi) * 4;
    s.vhi = vhi;
    tile_bases<NW, S>(s, d, state);
}

// Issue order of a tile's loads: for each of the kVecPerLane pieces, the S
// state arrays (W first), then the gradients in worker order; kTileLoads
// loads per tile.  A wave keeps a window of loads in flight beyond the one
// it waits for, and the window runs on into the wave's next tile.  Load j
// of a tile sits in ring slot j mod R; where the ring R does not divide the
// tile's loads, consecutive tiles take turns (phases) so that every load
// keeps its slot.  The depth follows the state policy (measured on MI355X):
//  - non-temporal state: a ring of 6 loads (five ahead), or 5 or 8 for a
//    few worker counts and optimizers (kRingTable), from a sweep of rings 4
//    to 8 for every worker count and optimizer (fraction of peak with
//    nothing cached, ResNet-269-shaped keys).  Six beats four everywhere
//    (momentum with 16 workers 0.765 against 0.717, plain SGD with 16 0.834
//    against 0.736, Adam with 10 0.731 against 0.673); eight is better for
//    Adam with 3-7 workers (3 workers: 0.752 against 0.684) and plain SGD
//    with 2, 3 or 6; five for momentum with 3 or 8 workers (8: 0.749
//    against 0.737).  Deeper windows flood the memory system with open
//    streams, and loads and stores share one in-order counter, so a load
//    issued after a state store is consumed only once that store has
//    completed;
//  - state held in the memory-side cache: a whole tile ahead (every load of
//    the next tile in flight while this one is consumed), since only the
//    gradient streams then reach HBM.
template <int NW, int S>
constexpr int kTileLoads = kVecPerLane * (NW + S);

// Ring of the non-temporal window, [S - 1][N - 1] (S = 1 plain SGD, 2
// momentum, 3 Adam): 6 unless another ring measured more than half a point
// better (momentum with 8 workers took 5 before its state was written back
// in the write phases below; with them, 6 is 5 points faster on a
// 143.7 M-parameter job).  A ring of 5 must divide the tile's 4 (N + S)
// loads; 6 and 8 take at most three and two phases.
constexpr int kRingTable[3][kMaxFixedWorkers] = {
    {6, 8, 8, 6, 6, 8, 6, 6, 6, 6, 6, 6, 6, 6, 6, 6},
    {6, 6, 5, 6, 6, 6, 6, 6, 6, 6, 6, 6, 6, 6, 6, 6},
    {6, 6, 8, 8, 8, 8, 8, 6, 6, 6, 6, 6, 6, 6, 6, 6},
};

#ifdef PHUB_LOADS_AHEAD
template <int NW, int S>
constexpr int kShallowAhead = PHUB_LOADS_AHEAD;  // a fixed depth, for sweeps
#else
template <int NW, int S>
constexpr int kShallowAhead =
    (NW >= 1 && NW <= kMaxFixedWorkers && S >= 1 && S <= 3 ? kRingTable[S - 1][NW - 1] : 6) - 1;
#endif

constexpr int gcd_int(int a, int b) { return b == 0 ? a : gcd_int(b, a % b); }

// Ring of the resident bin: a whole tile while that fits the registers
// (up to 80 loads, 320 VGPRs); beyond, the largest of 32, 24, 20, 16 loads
// that needs at most three phases (rings of 12 or 24 measured equal to the
// whole tile at 8-16 workers).
constexpr int resident_ring(int loads) {
    if (loads <= 80) return loads;
    for (int r : {32, 24, 20, 16})
        if (r / gcd_int(loads, r) <= 3) return r;
    return 4;
}

template <int NW, int S, bool RES>
constexpr int kAhead = RES ? resident_ring(kTileLoads<NW, S>) - 1 : kShallowAhead<NW, S>;

template <int NW, int S, bool RES>
constexpr int kRing = kAhead<NW, S, RES> + 1;

// Where the ring does not divide the tile's loads, a wave's tiles take
// kPhases turns: load j of a tile in phase h sits in ring slot
// (h L + j) mod R, and after kPhases tiles the slots line up again.
template <int NW, int S, bool RES>
constexpr int kPhases = kRing<NW, S, RES> / gcd_int(kTileLoads<NW, S>, kRing<NW, S, RES>);

// Burst write-back of the streamed bin's state, in chip-wide write phases.
// A few write streams spread evenly through many read streams cost HBM much
// more than the same bytes written in runs.  So, from enough workers per
// state array (burst_write_back), the streamed bin does not write a piece's
// new state as soon as it is computed: the state goes to a stash in LDS,
// and the wave writes the stash back in one run of stores when it finishes
// a piece inside the write window (then the tiles before the current one;
// at a tile's end, the tile too), or when the stash is full (kStashTiles
// tiles), or after its last tile.  The write window is the first part of a
// period of the device's constant-rate wall clock, which every wave of
// every launch on the chip reads alike: the waves write at the same time
// and read at the same time, so HBM sees long runs of writes and long runs
// of reads instead of a steady mix.  The period follows the tile's bytes
// and the stash's size (kWritePeriodNsPerStreamTile: about as many tiles of
// a wave as the stash holds besides the one in progress) and the window is
// about one tile long (kWriteWindowNs).  Measured on MI355X with
// nothing cached, fraction of peak (8 workers, momentum), piece by piece ->
// burst write-back: 143.7 M parameters 0.72 -> 0.815, 61.1 M 0.78 -> 0.816,
// 102 M with 16 workers 0.77 -> 0.84; the same stash flushed only when
// full, 0.73 on the first; flushed on each compute unit's own cycle counter
// (not aligned across the chip), 0.71; looked for only at the end of a tile
// (with the best period and window for that), 1-2.6 points below.
// Each lane reads back only the values it wrote, so the stash needs no
// barrier, and results do not depend on when it is written back.  The
// stash takes the compute unit's 160 KB of LDS (at most 40 KB per wave).
constexpr int kLdsBytes = 160 * 1024;
static_assert(kStashBytesPerWave * kWavesPerBlock <= kLdsBytes, "the stash fits the LDS");

template <int S>
constexpr int kStashTiles = stash_tiles(S);
static_assert(kVecPerLane * 1024 == 4 * 1024, "a tile is 4 KB per array and wave");

// float4 per tile and per wave in the stash (lane l holds entry l of every 64)
template <int S>
constexpr int kStashTileVecs = S * kVecPerLane * 64;

template <int NW, int S, bool RES, bool PULL>
constexpr bool kStash =
    !RES && !PULL && burst_write_back(NW, S) && kStashTiles<S> >= 2;


template <int NW, int S, bool RES, int I>
__device__ __forceinline__ f4 tile_load(const TileStreams<NW, S>& s) {
    constexpr int k = I % (NW + S);
    constexpr uint32_t o = uint32_t(I / (NW + S)) * 1024u;
    if constexpr (k < S)
        return load_wm<RES>(s.st[k], s.off + o);
    else
        return load_stream(s.g[k - S], s.off + o);
}

template <int NW, int S, bool RES>
struct TilePipe {
    static constexpr int R = kRing<NW, S, RES>;
    f4 ring[R];               // loads in flight, load j of a tile in slot j % R
    f4 acc[kVecPerLane];      // running gradient sums
    f4 sv[S][kVecPerLane];    // the state of each piece
};

// Writes back the stashed state of the wave's tiles [t0, t1] (streamed
// bin), tile by tile, each tile's S arrays piece by piece; tile t's state
// is in stash slot t mod kStashTiles.  `stash` points at the lane's entry
// of the wave's first stash slot.
template <int NW, int S>
__device__ __forceinline__ void write_stash(const DevTile* __restrict__ tiles, int32_t t0,
                                            int32_t t1, const PHUB_LDS f4* stash,
                                            float* const* state) {
    for (int32_t t = t0; t <= t1; ++t) {
        TileStreams<NW, S> s;
        tile_bases<NW, S>(s, tiles[t], state);
        const PHUB_LDS f4* ts = stash + (t % kStashTiles<S>) * kStashTileVecs<S>;
#pragma unroll
        for (int i = 0; i < S; ++i) {
#pragma unroll
            for (int u = 0; u < kVecPerLane; ++u) {
                const f4 v = ts[(i * kVecPerLane + u) * 64];
                store_wb(s.st[i], s.off + u * 1024u, v);
            }
        }
    }
}

// Where a wave's walk over a list of tiles stands in the burst write-back:
// tile t's state goes to stash slot t mod kStashTiles, and the tiles
// [t_stash, t) before the current one t wait in the stash.
struct TileCursor {
    const DevTile* tiles;
    PHUB_LDS f4* stash;  // the lane's entry of the wave's first slot
    int32_t t;
    int32_t t_stash;
    __device__ bool waiting() const { return t != t_stash; }
    // write back the tiles before the current one
    template <int NW, int S>
    __device__ void write_back_before(float* const* state) {
        write_stash<NW, S>(tiles, t_stash, t - 1, stash, state);
        t_stash = t;
    }
};

// Step I of a tile: issue load I + kAhead (of this tile, or of the next one
// if there is one), then consume load I.  After the last gradient of a
// piece, that piece is optimized and written back.  Just before the first
// load of the next tile is issued, the next tile's streams are formed from
// its descriptor and pointer row, which were fetched at the start of this
// tile.
template <int NW, int OPT, bool RES, bool PULL, int PH, int I, typename Cursor>
__device__ __forceinline__ void tile_step(TilePipe<NW, kStates<OPT>, RES>& p,
                                          const TileStreams<NW, kStates<OPT>>& a,
                                          TileStreams<NW, kStates<OPT>>& b, const DevTile& nd,
                                          uint64_t nrow, uint64_t prow, bool has_next,
                                          float* const* state, OptArgs o,
                                          PHUB_LDS f4* tile_stash, Cursor* cur) {
    constexpr int S = kStates<OPT>;
    constexpr int L = kTileLoads<NW, S>;
    constexpr int R = kRing<NW, S, RES>;
    constexpr int J = I + kAhead<NW, S, RES>;
    constexpr int base = (PH * L) % R;  // slot of this tile's first load
    if constexpr (J < L) {
        p.ring[(base + J) % R] = tile_load<NW, S, RES, J>(a);
    } else {
        if constexpr (J == L) tile_streams<NW, S>(b, nd, nrow, state);
        if (has_next) p.ring[(base + J) % R] = tile_load<NW, S, RES, J - L>(b);
    }
    __builtin_amdgcn_sched_barrier(0);
    const f4 v = p.ring[(base + I) % R];
    constexpr int k = I % (NW + S);
    constexpr int u = I / (NW + S);
    if constexpr (k < S)
        p.sv[k][u] = v;
    else if constexpr (k == S)
        p.acc[u] = v;
    else
        p.acc[u] = p.acc[u] + v;
    // Keep the addition (and so the wait for load I) at this step: the
    // compiler would otherwise sink the additions of the last piece past the
    // next-tile branch to their use, and issue that piece's loads as a burst.
    if constexpr (k > S) asm volatile("" : "+v"(p.acc[u]));
    if constexpr (k == NW + S - 1) {
        f4 st[S];
#pragma unroll
        for (int i = 0; i < S; ++i) st[i] = p.sv[i][u];
        update4<OPT>(p.acc[u], st, o);
        if constexpr (kStash<NW, S, RES, PULL>) {
#pragma unroll
            for (int i = 0; i < S; ++i) tile_stash[(i * kVecPerLane + u) * 64] = st[i];
            // the window opened during this tile: write back the tiles
            // before it now (this tile's pieces stay in its slot), so that
            // the waves' write-backs start within a piece of the window's
            // opening instead of within a tile
            if constexpr (u + 1 < kVecPerLane) {
                if (cur->waiting() && in_write_window(o.wb_period, o.wb_window))
                    cur->template write_back_before<NW, S>(state);
            }
        } else {
#pragma unroll
            for (int i = 0; i < S; ++i) store_wm<RES>(a.st[i], a.off + u * 1024u, st[i]);
        }
        if constexpr (PULL) {
            // the piece of w' into every worker's model buffer (pushpull)
#pragma unroll
            for (int w = 0; w < NW; ++w)
                store_out(const_cast<float*>(lane_pointer(prow, w)) + size_t(a.vhi) * 4,
                          a.off + u * 1024u, st[0]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int NW, int OPT, bool RES, bool PULL, int PH, typename Cursor, int... I>
__device__ __forceinline__ void tile_steps(std::integer_sequence<int, I...>,
                                           TilePipe<NW, kStates<OPT>, RES>& p,
                                           const TileStreams<NW, kStates<OPT>>& a,
                                           TileStreams<NW, kStates<OPT>>& b, const DevTile& nd,
                                           uint64_t nrow, uint64_t prow, bool has_next,
                                           float* const* state, OptArgs o,
                                           PHUB_LDS f4* tile_stash, Cursor* cur) {
    (tile_step<NW, OPT, RES, PULL, PH, I>(p, a, b, nd, nrow, prow, has_next, state, o, tile_stash,
                                          cur),
     ...);
}

template <int NW, int S, bool RES, int... I>
__device__ __forceinline__ void tile_prologue(std::integer_sequence<int, I...>,
                                              TilePipe<NW, S, RES>& p,
                                              const TileStreams<NW, S>& a) {
    ((p.ring[I % kRing<NW, S, RES>] = tile_load<NW, S, RES, I>(a)), ...);
}

// ------------------------------------------------------ the tile pool

// Dynamic schedule (work stealing): the streamed bin's full tiles of a
// launch form one pool, in address order, and every wave takes its next
// tile of the pool from a counter shared with the other waves of its XCD
// (PoolCounters), each counter serving every C-th tile, so that all waves
// still work on neighbouring tiles.  A wave that starts late (its compute
// unit was still held by another tenant's launch) simply takes fewer
// tiles.  A counter is never reset: the host passes each launch the
// counter's value at its start (the base), and every wave stops after
// exactly one take past its tiles.
//
// A take is a vector atomic from lane 0 whose value is read one tile later
// (issue_take, then resolve_take), so that the wait for it falls behind
// loads the wave has issued meanwhile, not in front of them.
__device__ __forceinline__ uint64_t issue_take(unsigned long long* counter) {
    uint64_t v = 0;
    if ((threadIdx.x & 63u) == 0) v = atomicAdd(counter, 1ull);
    return v;
}

// Pool index of a take, or -1 past the pool (or before it: never, unless
// the base is wrong, in which case nothing is read).
__device__ __forceinline__ int32_t resolve_take(uint64_t v, uint64_t base, int32_t count) {
    const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v))));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v >> 32))));
    const int64_t i = int64_t(((uint64_t(hi) << 32) | lo) - base);
    return i >= 0 && i < int64_t(count) ? int32_t(i) : -1;
}

// Writes back the `count` stashed tiles of a pool walk whose oldest sits in
// stash slot `first`, the next ones in the slots after it (mod SLOTS);
// slot k holds pool tile pool[idx[k] * stride].
template <int NW, int S, int SLOTS>
__device__ __forceinline__ void write_stash_slots(const DevTile* __restrict__ pool, int stride,
                                                  const int32_t (&idx)[SLOTS], int first,
                                                  int count, const PHUB_LDS f4* stash,
                                                  float* const* state) {
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
        if ((k - first + SLOTS) % SLOTS < count) {
            TileStreams<NW, S> s;
            tile_bases<NW, S>(s, pool[int64_t(idx[k]) * stride], state);
            const PHUB_LDS f4* ts = stash + k * kStashTileVecs<S>;
#pragma unroll
            for (int i = 0; i < S; ++i) {
#pragma unroll
                for (int u = 0; u < kVecPerLane; ++u) {
                    const f4 v = ts[(i * kVecPerLane + u) * 64];
                    store_wb(s.st[i], s.off + u * 1024u, v);
                }
            }
        }
    }
}

// Where a wave's pool walk stands in the burst write-back: its n-th tile
// (counted from 0) goes to stash slot n mod SLOTS, and the tiles
// [first, n) before the current one wait in the stash.
template <int SLOTS>
struct PoolCursor {
    const DevTile* pool;
    int stride;
    PHUB_LDS f4* stash;
    int32_t idx[SLOTS];  // the pool tile held by each slot
    int32_t n;
    int32_t first;
    __device__ bool waiting() const { return n != first; }
    // write back the tiles [first, end)
    template <int NW, int S>
    __device__ void write_back_to(int32_t end, float* const* state) {
        write_stash_slots<NW, S, SLOTS>(pool, stride, idx, first % SLOTS, end - first, stash,
                                        state);
        first = end;
    }
    template <int NW, int S>
    __device__ void write_back_before(float* const* state) {
        write_back_to<NW, S>(n, state);
    }
};

// ------------------------------------------------------------ remainders

// A remainder of a segment: nvec float4 and then rem (< 4) single elements
// per array.  Every lane's loads of a group of up to kVecPerLane float4 per
// array (as many as keep at most 64 loads in flight) and of its single
// element are issued before the first is consumed: a remainder shorter
// than a tile (the schedule's) costs one trip to memory, not one per
// float4 of a lane.
template <int NW, int OPT, bool RES, bool PULL>
__device__ __forceinline__ void partial(const float* const* g, float* const* stb,
                                        float* const* out, uint32_t nvec, uint32_t rem,
                                        OptArgs o) {
    constexpr int S = kStates<OPT>;
    constexpr int kGroup = (NW + S) * kVecPerLane <= 64 ? kVecPerLane
                           : 64 / (NW + S) > 0 ? 64 / (NW + S) : 1;
    const uint32_t lane = threadIdx.x & 63u;
    // the single elements of the last < 4, loaded with the first group
    const int64_t ti = int64_t(nvec) * 4 + lane;
    const bool tail = lane < rem;
    float ta[NW], tst[S];
    bool tail_loaded = false;
    for (uint32_t v0 = 0; v0 < nvec || !tail_loaded; v0 += 64u * kGroup) {
        f4 a[kGroup][NW];
        f4 st[kGroup][S];
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const uint32_t v = v0 + 64u * j + lane;
            if (v < nvec) {
#pragma unroll
                for (int w = 0; w < NW; ++w) a[j][w] = load_stream(g[w], v * 16u);
#pragma unroll
                for (int i = 0; i < S; ++i) st[j][i] = load_wm<RES>(stb[i], v * 16u);
            }
        }
        if (!tail_loaded && tail) {
#pragma unroll
            for (int w = 0; w < NW; ++w) ta[w] = load1(g[w], ti);
#pragma unroll
            for (int k = 0; k < S; ++k) tst[k] = load1(stb[k], ti);
        }
        tail_loaded = true;
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const uint32_t v = v0 + 64u * j + lane;
            if (v < nvec) {
                f4 s = a[j][0];
#pragma unroll
                for (int w = 1; w < NW; ++w) s = s + a[j][w];
                update4<OPT>(s, st[j], o);
#pragma unroll
                for (int i = 0; i < S; ++i) store_wm<RES>(stb[i], v * 16u, st[j][i]);
                if constexpr (PULL) {
#pragma unroll
                    for (int w = 0; w < NW; ++w) store_out(out[w], v * 16u, st[j][0]);
                }
            }
        }
    }
    if (tail) {
        float s = ta[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) s = s + ta[w];
        update<OPT>(s, tst, o);
#pragma unroll
        for (int k = 0; k < S; ++k) store1(stb[k], ti, tst[k]);
        if constexpr (PULL) {
#pragma unroll
            for (int w = 0; w < NW; ++w) store1(out[w], ti, tst[0]);
        }
    }
}

// The full tiles [tb, te) of one bin, NW workers, state policy RES; `first`
// is tiles[tb], which the wave has from its head.  At
// the start of tile t the wave fetches the pointer row of tile t + 1 (one
// vector load), whose descriptor it fetched at the start of tile t - 1, and
// the descriptor of tile t + 2 (a scalar load); both have long arrived when
// the window reaches tile t + 1.
template <int NW, int OPT, bool RES, bool PULL>
__device__ __forceinline__ void walk_tiles(const DevTile* __restrict__ tiles, int32_t tb,
                                           int32_t te, const DevTile& first,
                                           const float* const* __restrict__ grads,
                                           float* const* __restrict__ outs, float* const* state,
                                           OptArgs o, PHUB_LDS f4* stash) {
    constexpr int S = kStates<OPT>;
    constexpr int NPH = kPhases<NW, S, RES>;
    static_assert(NPH >= 1 && NPH <= 3, "the tile loop below unrolls at most three phases");
    if (tb >= te) return;
    const int32_t last = te - 1;
    TilePipe<NW, S, RES> p;
    TileStreams<NW, S> a, b;
    uint64_t prow = 0;  // pushpull: model-buffer pointer row of the current tile
    tile_streams<NW, S>(a, first, grads + int64_t(first.key) * NW, state);
    if constexpr (PULL) prow = load_row<NW>(outs + int64_t(first.key) * NW);
    DevTile nd = tiles[tb + 1 <= last ? tb + 1 : last];
    tile_prologue<NW, S, RES>(std::make_integer_sequence<int, kAhead<NW, S, RES>>{}, p, a);
    TileCursor c{tiles, stash, tb, tb};  // c.t: the current tile
    int32_t& t = c.t;
    // Tile t in ring phase PH; false after the bin's last tile.
    auto one_tile = [&](auto phase) -> bool {
        constexpr int PH = decltype(phase)::value;
        const bool has_next = t < last;
        const uint64_t nrow = load_row<NW>(grads + int64_t(nd.key) * NW);
        uint64_t nprow = 0;
        if constexpr (PULL) nprow = load_row<NW>(outs + int64_t(nd.key) * NW);
        const DevTile nd2 = tiles[t + 2 <= last ? t + 2 : last];
        PHUB_LDS f4* tile_stash = nullptr;  // this tile's slot of the stash
        if constexpr (kStash<NW, S, RES, PULL>)
            tile_stash = stash + (t % kStashTiles<S>) * kStashTileVecs<S>;
        tile_steps<NW, OPT, RES, PULL, PH>(std::make_integer_sequence<int, kTileLoads<NW, S>>{}, p,
                                           a, b, nd, nrow, prow, has_next, state, o, tile_stash,
                                           &c);
        if constexpr (kStash<NW, S, RES, PULL>) {
            if (t - c.t_stash == kStashTiles<S> - 1 || !has_next ||
                in_write_window(o.wb_period, o.wb_window)) {
                write_stash<NW, S>(tiles, c.t_stash, t, stash, state);
                c.t_stash = t + 1;
            }
        }
        if (!has_next) return false;
        a = b;
        nd = nd2;
        prow = nprow;
        ++t;
        return true;
    };
    for (;;) {
        if (!one_tile(std::integral_constant<int, 0>{})) break;
        if constexpr (NPH >= 2)
            if (!one_tile(std::integral_constant<int, 1 % NPH>{})) break;
        if constexpr (NPH >= 3)
            if (!one_tile(std::integral_constant<int, 2 % NPH>{})) break;
    }
}

// The streamed full tiles of a launch taken from its pool (dynamic
// schedule), NW workers: walk_tiles' pipeline, with the next tiles known
// from takes instead of a fixed list.  The wave's counter serves the pool
// tiles pool[i * stride], i < count.  At the start of tile t the wave
// resolves the take of tile t + 2 (issued at the start of tile t - 1),
// fetches that tile's descriptor and issues the take of tile t + 3 (only
// while takes still land in the pool).
template <int NW, int OPT, bool PULL>
__device__ __forceinline__ void walk_pool(const DevTile* __restrict__ pool, int32_t count,
                                          int stride, unsigned long long* counter, uint64_t base,
                                          const float* const* __restrict__ grads,
                                          float* const* __restrict__ outs, float* const* state,
                                          OptArgs o, PHUB_LDS f4* stash) {
    constexpr bool RES = false;
    constexpr int S = kStates<OPT>;
    constexpr int NPH = kPhases<NW, S, RES>;
    static_assert(NPH >= 1 && NPH <= 3, "the tile loop below unrolls at most three phases");
    constexpr bool STASH = kStash<NW, S, RES, PULL>;
    constexpr int SLOTS = STASH ? kStashTiles<S> : 1;
    int32_t cur = resolve_take(issue_take(counter), base, count);
    if (cur < 0) return;
    int32_t n1 = resolve_take(issue_take(counter), base, count);
    bool take2 = n1 >= 0;  // a take of the tile after next is in flight
    uint64_t v2 = take2 ? issue_take(counter) : 0;
    TilePipe<NW, S, RES> p;
    TileStreams<NW, S> a, b;
    uint64_t prow = 0;
    {
        const DevTile first = pool[int64_t(cur) * stride];
        tile_streams<NW, S>(a, first, grads + int64_t(first.key) * NW, state);
        if constexpr (PULL) prow = load_row<NW>(outs + int64_t(first.key) * NW);
    }
    DevTile nd = pool[int64_t(n1 >= 0 ? n1 : cur) * stride];
    tile_prologue<NW, S, RES>(std::make_integer_sequence<int, kAhead<NW, S, RES>>{}, p, a);
    PoolCursor<SLOTS> c{pool, stride, stash, {}, 0, 0};  // burst write-back
    auto one_tile = [&](auto phase) -> bool {
        constexpr int PH = decltype(phase)::value;
        const bool has_next = n1 >= 0;
        const uint64_t nrow = load_row<NW>(grads + int64_t(nd.key) * NW);
        uint64_t nprow = 0;
        if constexpr (PULL) nprow = load_row<NW>(outs + int64_t(nd.key) * NW);
        const int32_t n2 = take2 ? resolve_take(v2, base, count) : -1;
        const bool take3 = n2 >= 0;
        const uint64_t v3 = take3 ? issue_take(counter) : 0;
        const DevTile nd2 = pool[int64_t(n2 >= 0 ? n2 : cur) * stride];
        PHUB_LDS f4* tile_stash = nullptr;  // this tile's slot of the stash
        if constexpr (STASH) {
            const int sl = c.n % SLOTS;
            tile_stash = stash + sl * kStashTileVecs<S>;
#pragma unroll
            for (int k = 0; k < SLOTS; ++k)
                if (k == sl) c.idx[k] = cur;
        }
        tile_steps<NW, OPT, RES, PULL, PH>(std::make_integer_sequence<int, kTileLoads<NW, S>>{}, p,
                                           a, b, nd, nrow, prow, has_next, state, o, tile_stash,
                                           &c);
        if constexpr (STASH) {
            ++c.n;
            if (c.n - c.first == SLOTS || !has_next || in_write_window(o.wb_period, o.wb_window))
                c.template write_back_to<NW, S>(c.n, state);
        }
        if (!has_next) return false;
        a = b;
        nd = nd2;
        prow = nprow;
        cur = n1;
        n1 = n2;
        take2 = take3;
        v2 = v3;
        return true;
    };
    for (;;) {
        if (!one_tile(std::integral_constant<int, 0>{})) break;
        if constexpr (NPH >= 2)
            if (!one_tile(std::integral_constant<int, 1 % NPH>{})) break;
        if constexpr (NPH >= 3)
            if (!one_tile(std::integral_constant<int, 2 % NPH>{})) break;
    }
}

// The remainders [rb, re) of one bin; `first` is rems[rb], which the wave
// has from its head.  The descriptor of the next remainder is fetched while
// this one is processed.
template <int NW, int OPT, bool RES, bool PULL>
__device__ __forceinline__ void walk_rems(const DevRem* __restrict__ rems, int32_t rb, int32_t re,
                                          const DevRem& first,
                                          const float* const* __restrict__ grads,
                                          float* const* __restrict__ outs, float* const* state,
                                          OptArgs o) {
    constexpr int S = kStates<OPT>;
    DevRem rm = first;
    for (int32_t r = rb; r < re; ++r) {
        const DevRem next = rems[r + 1 < re ? r + 1 : r];
        const float* g[NW];
        float* out[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            g[w] = grads[int64_t(rm.key) * NW + w] + rm.offset;
            out[w] = PULL ? outs[int64_t(rm.key) * NW + w] + rm.offset : nullptr;
        }
        float* stb[S];
#pragma unroll
        for (int i = 0; i < S; ++i) stb[i] = state[i] + rm.arena_offset;
        partial<NW, OPT, RES, PULL>(g, stb, out, uint32_t(rm.count) >> 2,
                                    uint32_t(rm.count) & 3u, o);
        rm = next;
    }
}

}  // namespace

}  // namespace phub
