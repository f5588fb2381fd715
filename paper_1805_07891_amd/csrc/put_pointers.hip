// A small pointer table sent to the device as kernel arguments.
//
// Gradients in other buffers than the last step's (a backward pass that
// alternates between sets of buffers) change the pointer table every step.
// As a copy from a staging buffer that costs the stream a copy kernel and
// the handshake before it, and the host an event to track the buffer.  As
// the arguments of one launch the pointers are in the launch itself, and
// the host may change its table at once.  Measured (MI355X, a step with all
// pointers new, copy -> launch): 512 pointers over 2 M parameters 22.5 ->
// 19.3 us, 640 over 2.5 M 25.7 -> 22.6, 128 over 16 M 124.7 -> 120.9, 128
// over 0.8 M 11.1 -> 9.4 (bound by the host: 10.4 -> 8.9 us of it).  Two
// launches' worth of whole words took the 22.5 to 21.2 only, and three the
// host longer than the copy, so larger tables are copied.
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace phub {

namespace {

// (kernel arguments are limited to 4 KB: six bytes a pointer)
struct PutArgs {
    uint32_t lo[kPutPointers];
    uint16_t hi[kPutPointers];
};

__global__ __launch_bounds__(kPutPointers) void put_kernel(PutArgs a, uint64_t* __restrict__ dst,
                                                           int count) {
    const int i = int(threadIdx.x);
    if (i < count) dst[i] = (uint64_t(a.hi[i]) << 32) | a.lo[i];
}

}  // namespace

bool put_pointers(const void* const* pointers, size_t count, void* dst, hipStream_t stream,
                  hipError_t* error) {
    if (count > size_t(kPutPointers)) return false;
    PutArgs a;
    for (size_t i = 0; i < count; ++i) {
        const uint64_t p = reinterpret_cast<uint64_t>(pointers[i]);
        if (p >> 48) return false;  // no address of this GPU
        a.lo[i] = uint32_t(p);
        a.hi[i] = uint16_t(p >> 32);
    }
    hipLaunchKernelGGL(put_kernel, dim3(1), dim3(kPutPointers), 0, stream, a,
                       static_cast<uint64_t*>(dst), int(count));
    *error = hipGetLastError();
    return true;
}

}  // namespace phub
