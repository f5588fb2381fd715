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
#include "stream_walk.hpp"

namespace phub {

namespace {

// Loads of a block, and in flight.
constexpr int B = kManyBlock;
static_assert(kMaxFixedWorkers >= B, "every piece takes at least two blocks");

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
    walk_units<B, OPT, false>(tiles, h.tiles_streamed[0], h.tiles_streamed[1], grads, num_workers,
                           state, o, stash);
    walk_units<B, OPT, true>(tiles, h.tiles_resident[0], h.tiles_resident[1], grads, num_workers,
                             state, o, stash);
    walk_units<B, OPT, true>(rems, h.rems_resident[0], h.rems_resident[1], grads, num_workers,
                             state, o, stash);
    walk_units<B, OPT, false>(rems, h.rems_streamed[0], h.rems_streamed[1], grads, num_workers,
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
