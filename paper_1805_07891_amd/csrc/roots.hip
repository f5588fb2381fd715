// Check of the compiler's square root on the device: Adam's walks use it
// with and without the rounding check of sqrt_rn, so both must give the
// correctly rounded root for every fp32 value.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"

namespace {

constexpr int kRootThreads = 256, kRootGrid = 1024;

// Thread i takes the bit patterns i, i + threads, ... of all 2^32.  A double
// root rounded to fp32 is the correctly rounded fp32 root (53 bits are more
// than twice 24 and two).  wrong[0]: __builtin_sqrtf differs from it;
// wrong[1]: sqrt_rn does (any NaN is equal to any other).
__global__ __launch_bounds__(kRootThreads) void check_roots(unsigned long long* wrong) {
    uint32_t plain = 0, checked = 0;
    const uint64_t stride = uint64_t(kRootThreads) * kRootGrid;
    for (uint64_t b = uint64_t(blockIdx.x) * kRootThreads + threadIdx.x; b < (uint64_t(1) << 32);
         b += stride) {
        const float x = __builtin_bit_cast(float, uint32_t(b));
        double root = __builtin_sqrt(double(x));
        // (or the compiler would turn the three into one fp32 root)
        asm volatile("" : "+v"(root));
        const float want = float(root);
        const float p = __builtin_sqrtf(x), c = phub::sqrt_rn(x);
        const bool nan = want != want;
        plain += nan ? p == p : __builtin_bit_cast(uint32_t, p) != __builtin_bit_cast(uint32_t, want);
        checked += nan ? c == c : __builtin_bit_cast(uint32_t, c) != __builtin_bit_cast(uint32_t, want);
    }
    if (plain) atomicAdd(wrong, (unsigned long long)plain);
    if (checked) atomicAdd(wrong + 1, (unsigned long long)checked);
}

}  // namespace

// Enqueues the check on hip_stream.  wrong: device array of two counters,
// cleared by the caller; inputs where the compiler's root differs from the
// correctly rounded one are added to the first, those where sqrt_rn's does to
// the second.  Returns 0, -1 if wrong is NULL, or the HIP error code of the
// launch.
extern "C" int phub_check_roots(uint64_t* wrong, void* hip_stream) {
    if (!wrong) return -1;
    hipLaunchKernelGGL(check_roots, dim3(kRootGrid), dim3(kRootThreads), 0, (hipStream_t)hip_stream,
                       reinterpret_cast<unsigned long long*>(wrong));
    return int(hipGetLastError());
}
