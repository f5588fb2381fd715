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
// chip-wide write phases, as in tile_walk.hpp.  Measured (MI355X, 25.6 M
// parameters, momentum, nothing cached, fraction of 8 TB/s; before: batches
// of eight workers' loads issued together and drained, stores piece by
// piece): 17 workers 0.710 -> 0.821, 21 0.719 -> 0.841, 33 0.707 -> 0.855,
// 64 0.735 -> 0.844, 128 0.772 -> 0.840; Adam with 33 0.706 -> 0.827, plain
// SGD with 33 0.749 -> 0.849.  B = 6 was the best of 5 to 8 or within 0.7
// points of it at every count from 17 to 128 (5 up to 4 points below, 7 and
// 8 up to 2).
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "many_walk.hpp"

namespace phub {

namespace {

template <int OPT>
__global__ __launch_bounds__(kBlockThreads)
    __attribute__((amdgpu_waves_per_eu(1, 1))) void fused_step_many(PHUB_KERNEL_ARGS) {
    constexpr int T = stash_tiles(kStates<OPT>);
    __shared__ f4 stash_lds[kManyStash<T, OPT>];
    walk_many<T, OPT>(PHUB_MANY_ARGS, (PHUB_LDS f4*)stash_lds);
}

template <int OPT>
hipError_t launch(const StepParams& p, int grid, hipStream_t stream) {
    hipLaunchKernelGGL((fused_step_many<OPT>), dim3(grid), dim3(kBlockThreads), 0, stream,
                       PHUB_MANY_LAUNCH_ARGS);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fused_step_many(const StepParams& p, int optimizer, int grid,
                                  hipStream_t stream) {
    if (!many_takes(p)) return hipErrorInvalidValue;
    switch (optimizer) {
        case kOptMomentum: return launch<kOptMomentum>(p, grid, stream);
        case kOptNesterov: return launch<kOptNesterov>(p, grid, stream);
        case kOptSgd: return launch<kOptSgd>(p, grid, stream);
        case kOptAdam: return launch<kOptAdam>(p, grid, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace phub
