// The walk of the any-N stream kernels (fused_many.hip says what it does and
// why), for a stash of T tiles a wave.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"
#include "kernels.hpp"
#include "stream_walk.hpp"

namespace phub {

namespace {

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

// float4 of a workgroup's stash of T tiles a wave
template <int T, int OPT>
constexpr int kManyStash = kWavesPerBlock * T * kVecPerLane * kStates<OPT> * 64;

// A wave's whole work; stash_lds: the workgroup's stash.
template <int T, int OPT>
__device__ __forceinline__ void walk_many(PHUB_KERNEL_ARGS, PHUB_LDS f4* stash_lds) {
    constexpr int B = kManyBlock;
    static_assert(kMaxFixedWorkers >= B, "every piece takes at least two blocks");
    float* const state[3] = {weights, moments, second};
    const uint32_t wave = wave_index();
    constexpr int P = T * kVecPerLane;  // pieces of the stash
    PHUB_LDS f4* stash =
        stash_lds + (threadIdx.x >> 6) * (P * kStates<OPT> * 64) + (threadIdx.x & 63u);
    const WaveHead h = heads[wave];
    walk_units<B, OPT, false, P>(tiles, h.tiles_streamed[0], h.tiles_streamed[1], grads,
                                 num_workers, state, o, stash);
    walk_units<B, OPT, true, P>(tiles, h.tiles_resident[0], h.tiles_resident[1], grads,
                                num_workers, state, o, stash);
    walk_units<B, OPT, true, P>(rems, h.rems_resident[0], h.rems_resident[1], grads, num_workers,
                                state, o, stash);
    walk_units<B, OPT, false, P>(rems, h.rems_streamed[0], h.rems_streamed[1], grads, num_workers,
                                 state, o, stash);
    walk_ragged<OPT>(rems, h.rems_streamed[0], h.rems_streamed[1], grads, num_workers, state, o);
    walk_ragged<OPT>(rems, h.rems_resident[0], h.rems_resident[1], grads, num_workers, state, o);
}
#define PHUB_MANY_ARGS                                                                       \
    tiles, tile_begin, rems, rem_begin, heads, grads, outs, weights, moments, second, o,     \
        num_workers, pool, pool_count, pool_counters, pool_launch
#define PHUB_MANY_LAUNCH_ARGS                                                                \
    p.tiles, p.tile_begin, p.rems, p.rem_begin, p.heads, p.grads, p.outs, p.weights,         \
        p.moments, p.second, p.opt, p.num_workers, p.pool, p.pool_count, p.pool_counters,    \
        p.pool_launch

// Whether the any-N stream kernels can take a step.
inline bool many_takes(const StepParams& p) {
    // (a piece takes at least two blocks: the window's pointers run one ahead)
    return p.num_workers > kManyBlock && !p.outs && !p.merge && p.pool_count == 0;
}

}  // namespace

}  // namespace phub
