// The any-N stream kernel with a stash of at most 16 KB a wave, for steps
// whose state is cached (any_kernel in kernels.hpp): a compute unit's LDS
// then holds the workgroups of two or three launches.  (No limit of one wave
// per SIMD here either: the compiler would claim registers to enforce it.)
// The whole stash (40 KB) makes concurrent tenants' workgroups wait for each other's compute
// units, and gains nothing on jobs of few tiles.  Measured (MI355X, batches
// of fused_step_any -> whole stash -> this): 21 workers over 1 M parameters
// 21.9 -> 16.0 -> 16.1 us, four such jobs at once 65.5 -> 72.0 -> 65.6; Adam
// with 33 over 2 M 1.13 and 1.12 times faster, four at once 0.90 and 0.95.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "many_walk.hpp"

namespace phub {

namespace {

template <int OPT>
__global__ __launch_bounds__(kBlockThreads) void fused_step_many_shared(PHUB_KERNEL_ARGS) {
    constexpr int T = shared_stash_tiles(kStates<OPT>);
    __shared__ f4 stash_lds[kManyStash<T, OPT>];
    walk_many<T, OPT>(PHUB_MANY_ARGS, (PHUB_LDS f4*)stash_lds);
}

template <int OPT>
hipError_t launch(const StepParams& p, int grid, hipStream_t stream) {
    hipLaunchKernelGGL((fused_step_many_shared<OPT>), dim3(grid), dim3(kBlockThreads), 0, stream,
                       PHUB_MANY_LAUNCH_ARGS);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fused_step_many_shared(const StepParams& p, int optimizer, int grid,
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
