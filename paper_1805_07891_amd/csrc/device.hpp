// Device code shared by the kernels of the exchange step: the optimizers'
// arithmetic and the memory accesses (fused_step.hip, fused_many.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"

namespace phub {

typedef float f4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kWavesPerBlock = kBlockThreads / 64;

// ------------------------------------------------------------- optimizers

// State arrays of each optimizer, W first.
template <int OPT>
constexpr int kStates = OPT == kOptSgd ? 1 : (OPT == kOptAdam ? 3 : 2);

// Correctly rounded single-precision square root, with the rounding checked
// in double: the hardware root is within one ulp, the midpoints between
// neighbours have at most 25 significant bits, so their squares are exact in
// double and comparing x with them decides (a float's square root is never
// a midpoint, so there are no ties).  The compiler's own sequence for
// __builtin_sqrtf is correctly rounded too with the flag that the build
// sets, for all 2^32 inputs (roots.hip checks both), in half the
// instructions.  The streamed walk uses that (Adam with 16 and 33 workers
// +2.8 and +0.7 points); the piece-by-piece walks, whose load windows were
// tuned with the longer one, ran 0.3 to 3.6 points below without it (1 to 6
// workers, nothing cached, also with windows of 4, 6, 8 and 12 loads but
// for 3 and 4 workers), so they keep it.
__device__ __forceinline__ float sqrt_rn(float x) {
    const float y = __builtin_sqrtf(x);
    if (!(x > 0.0f) || !(y < __builtin_huge_valf())) return y;  // 0, < 0, NaN, inf
    const uint32_t yb = __builtin_bit_cast(uint32_t, y);
    const float down = __builtin_bit_cast(float, yb - 1u);
    const float up = __builtin_bit_cast(float, yb + 1u);
    const double lo = 0.5 * (double(down) + double(y));
    const double hi = 0.5 * (double(y) + double(up));
    const double xd = double(x);
    if (xd < lo * lo) return down;
    if (xd > hi * hi) return up;
    return y;
}

// One element: st[0] = w, st[1] = m, st[2] = v, updated in place.  CHECKED:
// with sqrt_rn's check (the same result either way).
template <int OPT, bool CHECKED = true>
__device__ __forceinline__ void update(float s, float* st, OptArgs o) {
    if constexpr (OPT == kOptSgd) {
        const float d = __builtin_fmaf(o.wd, st[0], s);
        st[0] = __builtin_fmaf(o.nlr, d, st[0]);
    } else if constexpr (OPT == kOptAdam) {
        const float d = __builtin_fmaf(o.wd, st[0], s);
        const float m = __builtin_fmaf(o.b1, st[1], o.c1 * d);
        const float dd = d * d;
        const float v = __builtin_fmaf(o.b2, st[2], o.c2 * dd);
        const float root = CHECKED ? sqrt_rn(v * o.k2) : __builtin_sqrtf(v * o.k2);
        const float den = root + o.eps;
        const float q = __fdiv_rn(o.k1 * m, den);
        st[0] = st[0] - q;
        st[1] = m;
        st[2] = v;
    } else {
        constexpr bool NEST = OPT == kOptNesterov;
        const float d = __builtin_fmaf(o.wd, st[0], s);
        const float m1 = __builtin_fmaf(o.mu, st[1], d);
        const float u = NEST ? __builtin_fmaf(o.mu, m1, d) : m1;
        st[0] = __builtin_fmaf(o.nlr, u, st[0]);
        st[1] = m1;
    }
}

// Four elements at once (a float4 of each array).
template <int OPT, bool CHECKED = true>
__device__ __forceinline__ void update4(const f4& s, f4* st, OptArgs o) {
    if constexpr (OPT == kOptAdam) {
        // the square root and division per component, correctly rounded
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float e[3] = {st[0][c], st[1][c], st[2][c]};
            update<OPT, CHECKED>(s[c], e, o);
            st[0][c] = e[0];
            st[1][c] = e[1];
            st[2][c] = e[2];
        }
    } else if constexpr (OPT == kOptSgd) {
        const f4 vwd = o.wd, vnlr = o.nlr;
        const f4 d = __builtin_elementwise_fma(vwd, st[0], s);
        st[0] = __builtin_elementwise_fma(vnlr, d, st[0]);
    } else {
        constexpr bool NEST = OPT == kOptNesterov;
        const f4 vwd = o.wd, vmu = o.mu, vnlr = o.nlr;
        const f4 d = __builtin_elementwise_fma(vwd, st[0], s);
        const f4 m1 = __builtin_elementwise_fma(vmu, st[1], d);
        const f4 u = NEST ? __builtin_elementwise_fma(vmu, m1, d) : m1;
        st[0] = __builtin_elementwise_fma(vnlr, u, st[0]);
        st[1] = m1;
    }
}

// --------------------------------------------------------- memory access

// Gradient pointers come from a table in memory, so the compiler cannot tell
// they address global memory and would emit flat loads (which wait on both
// the vector and the LDS counters).  Casting to the global address space
// gives global_load_dwordx4 with the uniform base in SGPRs and a 32-bit
// per-lane offset.
#define PHUB_GLOBAL __attribute__((address_space(1)))
#define PHUB_LDS __attribute__((address_space(3)))

// Gradient loads (and the unfused variant's sum buffer): non-temporal, as
// each gradient byte is read once.  A build with PHUB_GRADIENT_LOADS_CACHED
// set loads them cache-allocating instead: the ablation of caching the
// gradients beside the model (the paper's Table 4).
#ifndef PHUB_GRADIENT_LOADS_CACHED
#define PHUB_GRADIENT_LOADS_CACHED 0
#endif
__device__ __forceinline__ f4 load_stream(const float* base, uint32_t byte_off) {
    const PHUB_GLOBAL char* b = (const PHUB_GLOBAL char*)base;
#if PHUB_GRADIENT_LOADS_CACHED
    return *(const PHUB_GLOBAL f4*)(b + byte_off);
#else
    return __builtin_nontemporal_load((const PHUB_GLOBAL f4*)(b + byte_off));
#endif
}

// State accesses.  The policy is a template argument resolved with
// `if constexpr`: written as a run-time choice between two loads of the same
// address, the compiler merges the two loads into one and drops the
// non-temporal hint.
template <bool RES>
__device__ __forceinline__ f4 load_wm(const float* base, uint32_t byte_off) {
    const PHUB_GLOBAL f4* a = (const PHUB_GLOBAL f4*)((const PHUB_GLOBAL char*)base + byte_off);
    if constexpr (RES)
        return *a;
    else
        return __builtin_nontemporal_load(a);
}

template <bool RES>
__device__ __forceinline__ void store_wm(float* base, uint32_t byte_off, const f4& v) {
    PHUB_GLOBAL f4* a = (PHUB_GLOBAL f4*)((PHUB_GLOBAL char*)base + byte_off);
    if constexpr (RES)
        *a = v;
    else
        __builtin_nontemporal_store(v, a);
}

// A float4 of stashed state written back in a write phase: a buffer store
// (the compiler tracks it like any other store; the base in SGPRs, a 32-bit
// lane offset) with the cache policy bits of gfx950 given directly:
// non-temporal (2) with the sc1 bit (16).  Measured in the write phases
// against the non-temporal global store: +0.1 to +0.9 points on 8- and
// 16-worker jobs and +0.5 on four tenants; plain (cache-allocating) stores
// were 13-15 points below.  The descriptor covers 2 GB from the base, far
// beyond a tile's offsets (below 17 MB).
constexpr int kBufferWord3 = 0x00020000;  // buffer descriptor's format word on gfx9
constexpr int kWriteBackCachePolicy = 2 | 16;
__device__ __forceinline__ void store_wb(float* base, uint32_t byte_off, const f4& v) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, kBufferWord3);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, int(byte_off), 0, kWriteBackCachePolicy);
}

// Updated weights written to a worker's model buffer (pushpull): written
// once and not read by the step, so non-temporal.
__device__ __forceinline__ void store_out(float* base, uint32_t byte_off, const f4& v) {
    __builtin_nontemporal_store(v, (PHUB_GLOBAL f4*)((PHUB_GLOBAL char*)base + byte_off));
}

__device__ __forceinline__ float load1(const float* base, int64_t i) {
    return ((const PHUB_GLOBAL float*)base)[i];
}

__device__ __forceinline__ void store1(float* base, int64_t i, float v) {
    ((PHUB_GLOBAL float*)base)[i] = v;
}

__device__ __forceinline__ uint32_t wave_index() {
    return __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6));
}

// Whether the device's wall clock is inside a write window of the burst
// write-back (the same answer for every lane: the clock is a scalar).  The
// low 32 bits of the clock wrap every 43 s at 100 MHz; the wrap shifts the
// phase of the periods once, which costs nothing but a slightly misplaced
// window.
__device__ __forceinline__ bool in_write_window(uint32_t period, uint32_t window) {
    const uint32_t now = uint32_t(wall_clock64());
    return now % period < window;
}

// The kernel arguments are __restrict__: the schedule and the pointer table
// are never written by the kernel and the state never aliases the
// gradients, which lets the compiler fetch descriptors and pointers with
// scalar loads.
#define PHUB_KERNEL_ARGS                                                                  \
    const DevTile* __restrict__ tiles, const int32_t* __restrict__ tile_begin,            \
        const DevRem* __restrict__ rems, const int32_t* __restrict__ rem_begin,           \
        const WaveHead* __restrict__ heads,                                               \
        const float* const* __restrict__ grads, float* const* __restrict__ outs,          \
        float* __restrict__ weights, float* __restrict__ moments,                         \
        float* __restrict__ second, OptArgs o, int num_workers,                           \
        const DevTile* __restrict__ pool, int32_t pool_count,                             \
        unsigned long long* __restrict__ pool_counters, uint64_t pool_launch

// Splits a tile's float4 index into a part folded into the base pointers
// (a multiple of 2^20 float4, 16 MB) and a low part that keeps the per-lane
// 32-bit byte offset far from overflow.
constexpr uint32_t kVecLowMask = (1u << 20) - 1;

}  // namespace

}  // namespace phub
