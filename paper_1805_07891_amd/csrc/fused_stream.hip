// Fused aggregate + optimize kernels for the worker counts up to 32 with a
// kernel of their own in fused_step.hip, where walking the streamed tiles as
// one stream of load blocks (stream_walk.hpp) is faster than unrolling the
// window over a tile (stream_block in kernels.hpp says where, and the
// figures).  The cache-resident tiles and the remainders are walked as in
// fused_step.hip, by code of the same compile-time worker count: a
// remainder's loads all go out at once, and a resident tile's a tile ahead.
//
// The gain is in the write-back: it covers single pieces, so that at the
// window's opening nothing finished is held back for the rest of its tile,
// and it is looked for after every block; and, for Adam with 7 to 13
// workers, in having one at all.  (The worker count stays a run-time number
// in the stream walk: as a constant, the compiler peels its inner loop and
// waits for too many loads, 3 to 8 points down with blocks of 5.)
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"
#include "kernels.hpp"
#include "stream_walk.hpp"
#include "tile_walk.hpp"

namespace phub {

namespace {

template <int NW, int B, int OPT>
__global__ __launch_bounds__(kBlockThreads)
    __attribute__((amdgpu_waves_per_eu(1, 1))) void fused_step_stream(PHUB_KERNEL_ARGS) {
    static_assert(NW > B, "every piece takes at least two blocks");
    float* const state[3] = {weights, moments, second};
    const uint32_t wave = wave_index();
    constexpr int S = kStates<OPT>;
    constexpr int P = stash_tiles(S) * kVecPerLane;  // pieces of the stash
    __shared__ f4 stash_lds[kWavesPerBlock * P * S * 64];
    PHUB_LDS f4* stash = (PHUB_LDS f4*)stash_lds + (threadIdx.x >> 6) * (P * S * 64) +
                         (threadIdx.x & 63u);
    const WaveHead h = heads[wave];
    walk_units<B, OPT, false, P>(tiles, h.tiles_streamed[0], h.tiles_streamed[1], grads,
                                 num_workers, state, o, stash);
    walk_tiles<NW, OPT, true, false>(tiles, h.tiles_resident[0], h.tiles_resident[1],
                                     h.first_resident, grads, outs, state, o, nullptr);
    walk_rems<NW, OPT, true, false>(rems, h.rems_resident[0], h.rems_resident[1],
                                    h.first_rem_resident, grads, outs, state, o);
    walk_rems<NW, OPT, false, false>(rems, h.rems_streamed[0], h.rems_streamed[1],
                                     h.first_rem_streamed, grads, outs, state, o);
}

template <int NW, int OPT>
hipError_t launch(const StepParams& p, int grid, hipStream_t stream) {
    constexpr int B = stream_block(NW, kStates<OPT>);
    if constexpr (B > 0) {
        hipLaunchKernelGGL((fused_step_stream<NW, B, OPT>), dim3(grid), dim3(kBlockThreads), 0,
                           stream, p.tiles, p.tile_begin, p.rems, p.rem_begin, p.heads, p.grads,
                           p.outs, p.weights, p.moments, p.second, p.opt, p.num_workers, p.pool,
                           p.pool_count, p.pool_counters, p.pool_launch);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

}  // namespace

template <int OPT>
hipError_t launch_stream(const StepParams& p, int grid, hipStream_t stream) {
    if (p.outs || p.merge || p.pool_count > 0) return hipErrorInvalidValue;
    switch (p.num_workers) {
        case 7: return launch<7, OPT>(p, grid, stream);
        case 8: return launch<8, OPT>(p, grid, stream);
        case 9: return launch<9, OPT>(p, grid, stream);
        case 10: return launch<10, OPT>(p, grid, stream);
        case 11: return launch<11, OPT>(p, grid, stream);
        case 12: return launch<12, OPT>(p, grid, stream);
        case 13: return launch<13, OPT>(p, grid, stream);
        case 14: return launch<14, OPT>(p, grid, stream);
        case 15: return launch<15, OPT>(p, grid, stream);
        case 16: return launch<16, OPT>(p, grid, stream);
        case 20: return launch<20, OPT>(p, grid, stream);
        case 24: return launch<24, OPT>(p, grid, stream);
        case 32: return launch<32, OPT>(p, grid, stream);
        default: return hipErrorInvalidValue;
    }
}

// (as fused_step.hip: all optimizers, or one per part)
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 0
template hipError_t launch_stream<kOptMomentum>(const StepParams&, int, hipStream_t);
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 2
template hipError_t launch_stream<kOptNesterov>(const StepParams&, int, hipStream_t);
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 4
template hipError_t launch_stream<kOptSgd>(const StepParams&, int, hipStream_t);
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 6
template hipError_t launch_stream<kOptAdam>(const StepParams&, int, hipStream_t);
#endif

}  // namespace phub
