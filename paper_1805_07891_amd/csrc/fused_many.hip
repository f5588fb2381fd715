// Fused aggregate + optimize kernel of the exchange step for worker counts
// without a kernel of their own (17 and more; fused_step.hip has the
// others, and the steps that write model buffers).
//
// The work, the schedule and the arithmetic are fused_step.hip's: a wave
// walks its bins, the sum is a left fold in worker order, the optimizer
// runs in the same pass.  Here the worker count is a run-time number, so
// the load window cannot be unrolled over a tile.  Instead the wave's work
// is one sequence of blocks of B loads: for each piece (64 float4, 1 KB of
// every array) the workers in blocks of B, the last block filled up with
// loads of the last worker's first line that are not added.  B registers
// hold the loads in flight.  A step waits for load j of the current block,
// adds it, and issues load j of the next block into the same register, so
// that B loads are always in flight, across pieces and tiles, and the loop
// body is one block long whatever the worker count.  A block's gradient
// pointers are fetched one block ahead with one vector load.
//
// What bounds it is HBM, and most of all how its few writes are spread: the
// same loads without the state stores ran at 0.88-0.97 of peak, with a
// piece's stores issued as soon as it is done at 0.71-0.73, though they are
// 3-10% of the bytes.  So the tiles' state is written back in bursts in the
// chip-wide write phases, as in fused_step.hip.  Measured (MI355X, 25.6 M
// parameters, momentum, nothing cached, fraction of 8 TB/s; before: batches
// of eight workers' loads issued together and drained, stores piece by
// piece): 17 workers 0.710 -> 0.821, 21 0.719 -> 0.841, 33 0.707 -> 0.855,
// 64 0.735 -> 0.844, 128 0.772 -> 0.840; Adam with 33 0.706 -> 0.827, plain
// SGD with 33 0.749 -> 0.849.  B = 6 was the best of 5 to 8 or within 0.7
// points of it at every count from 17 to 128 (5 up to 4 points below, 7 and
// 8 up to 2).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"
#include "kernels.hpp"

namespace phub {

namespace {

// Loads of a block, and in flight.
constexpr int B = 6;
static_assert(kMaxFixedWorkers >= B, "every piece takes at least two blocks");

// One run of up to 256 float4 of a key: a full tile or a remainder's whole
// float4s.
struct Unit {
    const float* const* row;  // the key's gradient pointers
    int64_t base;             // element of the state arenas that byte offset 0 stands for
    uint32_t vlo;             // float4 index of the unit's first, beside vhi
    uint32_t vhi;             // float4 index folded into the gradient bases
    uint32_t nvec;
};

// The units of a bin: its full tiles (DevTile) or its remainders (DevRem;
// those shorter than a float4 have no unit), each descriptor fetched one
// unit before its own is decoded.
template <typename DESC>
struct UnitList {
    const DESC* desc;
    int32_t i, end;  // the fetched descriptor's index, the bin's end
    DESC d;

    __device__ __forceinline__ void fetch() {
        if constexpr (sizeof(DESC) == sizeof(DevRem))
            while (i < end && desc[i].count < 4) ++i;
        if (i < end) d = desc[i];
    }
    __device__ __forceinline__ UnitList(const DESC* all, int32_t b, int32_t e)
        : desc(all), i(b), end(e) {
        fetch();
    }
    __device__ __forceinline__ bool more() const { return i < end; }
    __device__ __forceinline__ const float* const* row(const float* const* grads, int n) const {
        return grads + int64_t(d.key) * n;
    }
    __device__ __forceinline__ Unit take(const float* const* grads, int n) {
        Unit u;
        uint64_t vec;
        if constexpr (sizeof(DESC) == sizeof(DevRem)) {
            vec = uint64_t(d.offset) / 4;
            u.nvec = uint32_t(d.count) >> 2;
        } else {
            vec = d.vec;
            u.nvec = uint32_t(kTileElems / 4);
        }
        u.vlo = uint32_t(vec) & kVecLowMask;
        u.vhi = uint32_t(vec) & ~kVecLowMask;
        u.base = d.arena_offset - int64_t(u.vlo) * 4;
        u.row = row(grads, n);
        ++i;
        fetch();
        return u;
    }
};

// Byte offset of the lane's float4 of piece u; lanes past the unit's end
// repeat its last float4.
__device__ __forceinline__ uint32_t lane_off(const Unit& c, uint32_t u) {
    const uint32_t v = u * 64u + (threadIdx.x & 63u);
    return (c.vlo + (v < c.nvec ? v : c.nvec - 1)) * 16u;
}

// Gradient bases of the block whose first worker is w0, lane j holding
// worker w0 + j's (past the last worker, the last one's): one vector load,
// issued one block before its first use, so that it returns with the data
// loads issued around it.
__device__ __forceinline__ uint64_t block_pointers(const float* const* row, int w0, int n) {
    const int l = int(threadIdx.x & 63u);
    const int w = w0 + (l < B ? l : B - 1);
    return ((const PHUB_GLOBAL uint64_t*)row)[uint32_t(w < n ? w : n - 1)];
}

__device__ __forceinline__ const float* lane_base(uint64_t p, int j) {
    const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(p)), j));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(p >> 32)), j));
    return reinterpret_cast<const float*>((uint64_t(hi) << 32) | lo);
}

// Burst write-back of the streamed tiles' state, as in fused_step.hip: a
// finished piece's state goes to a stash in LDS (kStashPieces pieces per
// wave, lane l holding entry l of every 64), and the wave writes the stash
// back in one run of stores when the chip-wide write window is open (looked
// at after every block of loads), when the stash is full, or after its last
// piece.  Each lane reads back only what it wrote: no barrier.
template <int S>
constexpr int kStashPieces = stash_tiles(S) * kVecPerLane;

template <int S>
struct Stash {
    PHUB_LDS f4* lds;  // the lane's entry of the wave's first piece
    uint32_t lo = 0;   // lane k: where piece k's state goes (element index
    uint32_t hi = 0;   // in the state arenas)
    int count = 0;

    __device__ __forceinline__ void put(const f4 (&st)[S], int64_t elem) {
        lo = lane == uint32_t(count) ? uint32_t(elem) : lo;
        hi = lane == uint32_t(count) ? uint32_t(uint64_t(elem) >> 32) : hi;
#pragma unroll
        for (int i = 0; i < S; ++i) lds[(count * S + i) * 64] = st[i];
        ++count;
    }
    template <bool RES>
    __device__ __forceinline__ void write_back(float* const* state) {
#pragma unroll
        for (int i = 0; i < S; ++i) {
            for (int k0 = 0; k0 < count; k0 += kVecPerLane) {
                f4 r[kVecPerLane];
#pragma unroll
                for (int k = 0; k < kVecPerLane; ++k) r[k] = lds[((k0 + k) * S + i) * 64];
#pragma unroll
                for (int k = 0; k < kVecPerLane; ++k) {
                    if (k0 + k < count) {
                        const uint32_t l = uint32_t(__builtin_amdgcn_readlane(int(lo), k0 + k));
                        const uint32_t h = uint32_t(__builtin_amdgcn_readlane(int(hi), k0 + k));
                        float* const a = state[i] + int64_t((uint64_t(h) << 32) | l);
                        if constexpr (RES)
                            store_wm<true>(a, lane * 16u, r[k]);
                        else
                            store_wb(a, lane * 16u, r[k]);
                    }
                }
            }
        }
        count = 0;
    }
    uint32_t lane = threadIdx.x & 63u;
};

template <int OPT, bool RES, typename DESC>
__device__ __forceinline__ void walk_units(const DESC* desc, int32_t begin, int32_t end,
                                           const float* const* grads, int n, float* const* state,
                                           OptArgs o, PHUB_LDS f4* stash_lds) {
    constexpr int S = kStates<OPT>;
    constexpr bool STASH = sizeof(DESC) == sizeof(DevTile);
    Stash<S> stash{stash_lds};
    UnitList<DESC> list(desc, begin, end);
    if (!list.more()) return;
    const int last = (n - 1) / B * B;  // first worker of the last block
    const int tail = n - last;         // its workers
    const uint32_t lane = threadIdx.x & 63u;
    Unit c = list.take(grads, n);
    f4 v[B];
    uint32_t u = 0;
    uint32_t off = lane_off(c, 0);
    uint64_t p = block_pointers(c.row, 0, n) + uint64_t(c.vhi) * 16u;
    uint64_t q = block_pointers(c.row, B, n);
#pragma unroll
    for (int j = 0; j < B; ++j) v[j] = load_stream(lane_base(p, j), off);
    f4 acc, st[S];
    auto load_state = [&]() {
#pragma unroll
        for (int i = 0; i < S; ++i) st[i] = load_wm<RES>(state[i] + c.base, off);
    };
    auto finish = [&](int64_t base, uint32_t vlo, uint32_t nvec, uint32_t u, uint32_t off) {
        update4<OPT>(acc, st, o);
        if constexpr (STASH) {
            stash.put(st, base + int64_t(vlo + u * 64u) * 4);
        } else if (u * 64u + lane < nvec) {
#pragma unroll
            for (int i = 0; i < S; ++i) store_wm<RES>(state[i] + base, off, st[i]);
        }
    };
    for (;;) {
        const bool same = (u + 1) * 64u < c.nvec;
        const bool has = same || list.more();
        acc = -0.0f;  // -0 + x is x, bit for bit
        // All but the last block: issue the next block of this piece.  p:
        // the bases of the block being issued; q: of the one after it.
        for (int w0 = 0; w0 < last; w0 += B) {
            if constexpr (STASH) {
                if (stash.count && (stash.count == kStashPieces<S> ||
                                    in_write_window(o.wb_period, o.wb_window)))
                    stash.template write_back<RES>(state);
            }
            p = q + uint64_t(c.vhi) * 16u;
            if (w0 + B < last)
                q = block_pointers(c.row, w0 + 2 * B, n);
            else
                q = block_pointers(same || !has ? c.row : list.row(grads, n), 0, n);
            // the loads of the next block past the last worker: one line only
            const int real = w0 + B < last ? B : tail;
            const uint32_t spare = uint32_t(__builtin_amdgcn_readfirstlane(int(off)));
#pragma unroll
            for (int j = 0; j < B; ++j) {
                acc = acc + v[j];
                asm volatile("" : "+v"(acc));  // keep the wait for load j here
                v[j] = load_stream(lane_base(p, j), j < real ? off : spare);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!has) break;
        // The last block: issue the piece's state loads, then the first
        // block of the next piece.
        load_state();
        const int64_t base = c.base;
        const uint32_t vlo = c.vlo, nvec = c.nvec, pu = u, poff = off;
        if (!same) c = list.take(grads, n);
        u = same ? u + 1 : 0;
        off = lane_off(c, u);
        p = q + uint64_t(c.vhi) * 16u;
        q = block_pointers(c.row, B, n);
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const f4 sum = acc + v[j];
            acc = j < tail ? sum : acc;
            asm volatile("" : "+v"(acc));
            v[j] = load_stream(lane_base(p, j), off);
            __builtin_amdgcn_sched_barrier(0);
        }
        finish(base, vlo, nvec, pu, poff);
        __builtin_amdgcn_sched_barrier(0);
    }
    // the last block of the last piece
    load_state();
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const f4 sum = acc + v[j];
        acc = j < tail ? sum : acc;
    }
    finish(c.base, c.vlo, c.nvec, u, off);
    if constexpr (STASH) stash.template write_back<RES>(state);
}

// The last 1-3 elements of each remainder of a bin.  Lane 4 k + e of a load
// takes element e of worker 16 i + k, so that 64 workers' loads go out
// together; the sum then folds them in worker order.
template <int OPT>
__device__ __forceinline__ void walk_ragged(const DevRem* __restrict__ rems, int32_t rb, int32_t re,
                                            const float* const* __restrict__ grads, int n,
                                            float* const* state, OptArgs o) {
    constexpr int S = kStates<OPT>;
    constexpr int G = 4;
    const int lane = int(threadIdx.x & 63u);
    const int e = lane & 3;
    for (int32_t r = rb; r < re; ++r) {
        const DevRem d = rems[r];
        const int ragged = d.count & 3;
        if (!ragged) continue;
        const int64_t done = d.count & ~3;
        const PHUB_GLOBAL uint64_t* row =
            (const PHUB_GLOBAL uint64_t*)grads + int64_t(d.key) * n;
        const bool mine = lane < ragged;
        float st[S];
        if (mine) {
#pragma unroll
            for (int i = 0; i < S; ++i) st[i] = load1(state[i], d.arena_offset + done + lane);
        }
        float s = -0.0f;
        for (int w0 = 0; w0 < n; w0 += 16 * G) {
            float x[G];
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const int w = w0 + 16 * i + (lane >> 2);
                x[i] = 0.0f;
                if (w < n && e < ragged)
                    x[i] = load1(reinterpret_cast<const float*>(row[w]), d.offset + done + e);
            }
#pragma unroll
            for (int i = 0; i < G; ++i)
                for (int k = 0; k < 16; ++k)
                    if (w0 + 16 * i + k < n) s = s + __shfl(x[i], 4 * k + e);
        }
        if (mine) {
            update<OPT>(s, st, o);
#pragma unroll
            for (int i = 0; i < S; ++i) store1(state[i], d.arena_offset + done + lane, st[i]);
        }
    }
}

template <int OPT>
__global__ __launch_bounds__(kBlockThreads)
    __attribute__((amdgpu_waves_per_eu(1, 1))) void fused_step_many(PHUB_KERNEL_ARGS) {
    float* const state[3] = {weights, moments, second};
    const uint32_t wave = wave_index();
    constexpr int S = kStates<OPT>;
    __shared__ f4 stash_lds[kWavesPerBlock * kStashPieces<S> * S * 64];
    PHUB_LDS f4* stash = (PHUB_LDS f4*)stash_lds +
                         (threadIdx.x >> 6) * (kStashPieces<S> * S * 64) + (threadIdx.x & 63u);
    const WaveHead h = heads[wave];
    walk_units<OPT, false>(tiles, h.tiles_streamed[0], h.tiles_streamed[1], grads, num_workers,
                           state, o, stash);
    walk_units<OPT, true>(tiles, h.tiles_resident[0], h.tiles_resident[1], grads, num_workers,
                             state, o, stash);
    walk_units<OPT, true>(rems, h.rems_resident[0], h.rems_resident[1], grads, num_workers,
                             state, o, stash);
    walk_units<OPT, false>(rems, h.rems_streamed[0], h.rems_streamed[1], grads, num_workers,
                              state, o, stash);
    walk_ragged<OPT>(rems, h.rems_streamed[0], h.rems_streamed[1], grads, num_workers, state, o);
    walk_ragged<OPT>(rems, h.rems_resident[0], h.rems_resident[1], grads, num_workers, state, o);
}

template <int OPT>
hipError_t launch(const StepParams& p, int grid, hipStream_t stream) {
    hipLaunchKernelGGL((fused_step_many<OPT>), dim3(grid), dim3(kBlockThreads), 0, stream,
                       p.tiles, p.tile_begin, p.rems, p.rem_begin, p.heads, p.grads, p.outs,
                       p.weights, p.moments, p.second, p.opt, p.num_workers, p.pool, p.pool_count,
                       p.pool_counters, p.pool_launch);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fused_step_many(const StepParams& p, int optimizer, int grid,
                                  hipStream_t stream) {
    // (a piece takes at least two blocks: the window's pointers run one ahead)
    if (p.num_workers <= B || p.outs || p.merge || p.pool_count > 0) return hipErrorInvalidValue;
    switch (optimizer) {
        case kOptMomentum: return launch<kOptMomentum>(p, grid, stream);
        case kOptNesterov: return launch<kOptNesterov>(p, grid, stream);
        case kOptSgd: return launch<kOptSgd>(p, grid, stream);
        case kOptAdam: return launch<kOptAdam>(p, grid, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace phub
