// Fused aggregate + optimize kernel of the exchange step, for gfx950.
//
// One wave plays the role of one PHub core (paper, section 3.2.4): it walks
// the list of chunks the schedule fixed for it at initialisation, and for
// each element it sums the N workers' gradients
// (section 3.2.2, "tall" aggregation: one worker takes the same chunk
// across all gradient arrays) and immediately runs the optimizer on that
// element (section 3.2.2: the thread that aggregates a chunk also
// optimizes it).  Waves never synchronise with each other.  The partial sum
// never leaves registers, so there is no merge buffer: each gradient byte is
// read once and each optimizer state array is read and written once.
//
// Optimizers are pluggable (section 3.2.2): momentum SGD (plain or
// Nesterov; state W, M), plain SGD (state W) and Adam (state W, M, V) are
// compile-time policies of the same kernel; the S state arrays stream
// beside the N gradients.
//
// Launch shape: one workgroup of kBlockThreads per compute unit, persistent.
// The step is HBM-bound and mixes many read streams with a few in-place
// write streams (the state); on MI355X such a mix reaches the highest
// bandwidth with few waves per CU.
//
// Memory access: a wave reads its head (its bins and the first descriptor
// of each, WaveHead), then walks its full tiles, then its remainders.  A
// tile is 1024 elements of each of the N + S arrays: a lane takes 4 float4
// of each (the wave's 64 lanes cover 4 contiguous 1 KB pieces).  Segments
// are cut on the host into full tiles and a remainder, so the tile loop is
// straight-line code.  The tile's loads go out piece by piece in a sliding
// window that continues into the wave's next tile (see the load window
// below); each piece is optimized as soon as its last gradient is in, and
// written back at once, or, from enough gradient streams per state stream,
// in bursts of several tiles through LDS, timed by a chip-wide clock so
// that all waves write together (the burst write-back below).  Gradients
// are read once per step and loaded non-temporally.  A wave has two bins:
// the part of the job whose state is read and written non-temporally like
// the gradients, and the part whose state stays in the memory-side cache
// between steps (cache-allocating loads and stores).  Either may be empty.
//
// Arithmetic (no MFMA: the work is elementwise and HBM-bound): the sum is a
// left fold in ascending worker index, plain fp32 additions; then the
// optimizer, e.g. for momentum four fused multiply-adds:
//     d = wd*w + s;  m' = mu*m + d;  u = mu*m' + d (Nesterov) or m';
//     w' = -lr*u + w.
// The file is compiled with -ffp-contract=off and without fast-math, so the
// compiler neither fuses nor reorders beyond the explicit fma calls, and
// subnormals are kept; Adam's square root and division are correctly
// rounded (the division by the compiler's IEEE sequence, the square root
// by sqrt_rn below).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"
#include "kernels.hpp"
#include "tile_walk.hpp"

namespace phub {

namespace {

// ---------------------------------------------------------------- kernels

// NW > 0: exactly NW workers.  Each wave streams the full tiles of its
// streamed bin, then those of its cache-resident bin, then the remainders
// of both.  All waves thus work in the same phase at almost every moment:
// on MI355X that measured better than mixing the two kinds of traffic
// (odd waves in the other order), and slightly better than the resident
// bin first.  One wave per SIMD (one workgroup of 4 waves per CU).
#define PHUB_ONE_WAVE_PER_SIMD __attribute__((amdgpu_waves_per_eu(1, 1)))

template <int NW, int OPT, bool PULL>
__global__ __launch_bounds__(kBlockThreads) PHUB_ONE_WAVE_PER_SIMD void fused_step_fixed(
    PHUB_KERNEL_ARGS) {
    float* const state[3] = {weights, moments, second};
    const uint32_t wave = wave_index();
    constexpr int S = kStates<OPT>;
    PHUB_LDS f4* stash = nullptr;  // the lane's entry of its wave's stash
    if constexpr (kStash<NW, S, false, PULL>) {
        __shared__ f4 stash_lds[kWavesPerBlock * kStashTiles<S> * kStashTileVecs<S>];
        stash = (PHUB_LDS f4*)stash_lds +
                (threadIdx.x >> 6) * (kStashTiles<S> * kStashTileVecs<S>) + (threadIdx.x & 63u);
    }
    // the wave's bins and the first descriptor of each, read at once
    const WaveHead h = heads[wave];
    if (pool_count > 0) {
        // this workgroup's counter, the pool tiles it serves, and the
        // counter's value at the start of this launch
        const int nc = pool_counter_count(gridDim.x);
        const int c = int(blockIdx.x % uint32_t(nc));
        const int64_t served = pool_counter_tiles(pool_count, c, nc);
        const uint64_t per_launch =
            uint64_t(served) + uint64_t(kWavesPerBlock) * uint64_t(pool_counter_groups(gridDim.x, c, nc));
        walk_pool<NW, OPT, PULL>(pool + c, int32_t(served), nc,
                                 pool_counters + c * kPoolCounterStride,
                                 pool_launch * per_launch, grads, outs, state, o, stash);
    } else {
        walk_tiles<NW, OPT, false, PULL>(tiles, h.tiles_streamed[0], h.tiles_streamed[1],
                                         h.first_streamed, grads, outs, state, o, stash);
    }
    walk_tiles<NW, OPT, true, PULL>(tiles, h.tiles_resident[0], h.tiles_resident[1],
                                    h.first_resident, grads, outs, state, o, stash);
    walk_rems<NW, OPT, true, PULL>(rems, h.rems_resident[0], h.rems_resident[1],
                                   h.first_rem_resident, grads, outs, state, o);
    walk_rems<NW, OPT, false, PULL>(rems, h.rems_streamed[0], h.rems_streamed[1],
                                    h.first_rem_streamed, grads, outs, state, o);
}

// Any N, the worker count a run-time number: workers taken in batches of
// kBatch, each batch's loads in flight together, the running sum carried
// across batches in worker order.  It takes the pushpull steps, and the other
// steps where any_kernel (kernels.hpp) says so; fused_many.hip has the rest.
constexpr int kBatch = 8;

__device__ __forceinline__ f4 sum_any(const float* const* kp, int n, int64_t offset,
                                      uint32_t bo) {
    f4 s = load_stream(kp[0] + offset, bo);
    for (int w0 = 1; w0 < n; w0 += kBatch) {
        f4 a[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (w0 + j < n) a[j] = load_stream(kp[w0 + j] + offset, bo);
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (w0 + j < n) s = s + a[j];
    }
    return s;
}

// The same over kVecPerLane float4 per lane at once (1 KB apart): every
// batch keeps kBatch * kVecPerLane loads in flight.
__device__ __forceinline__ void sum_any_pieces(const float* const* kp, int n, int64_t offset,
                                               uint32_t bo, f4* s) {
#pragma unroll
    for (int u = 0; u < kVecPerLane; ++u) s[u] = load_stream(kp[0] + offset, bo + u * 1024u);
    for (int w0 = 1; w0 < n; w0 += kBatch) {
        f4 a[kBatch][kVecPerLane];
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (w0 + j < n) {
#pragma unroll
                for (int u = 0; u < kVecPerLane; ++u)
                    a[j][u] = load_stream(kp[w0 + j] + offset, bo + u * 1024u);
            }
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (w0 + j < n) {
#pragma unroll
                for (int u = 0; u < kVecPerLane; ++u) s[u] = s[u] + a[j][u];
            }
    }
}

template <int OPT, bool RES, bool PULL>
__device__ __forceinline__ void run_any(const float* const* kp, float* const* ko, int n,
                                        int64_t offset, float* const* stb, uint32_t nvec,
                                        uint32_t rem, OptArgs o) {
    constexpr int S = kStates<OPT>;
    const uint32_t lane = threadIdx.x & 63u;
    // whole groups of kVecPerLane * 64 float4 (a full tile is one), then the rest
    const uint32_t nfull = nvec / (64u * kVecPerLane) * (64u * kVecPerLane);
    for (uint32_t v = lane; v < nfull; v += 64u * kVecPerLane) {
        const uint32_t bo = v * 16u;
        f4 sum[kVecPerLane];
        sum_any_pieces(kp, n, offset, bo, sum);
        f4 st[kVecPerLane][S];
#pragma unroll
        for (int u = 0; u < kVecPerLane; ++u)
#pragma unroll
            for (int i = 0; i < S; ++i) st[u][i] = load_wm<RES>(stb[i], bo + u * 1024u);
#pragma unroll
        for (int u = 0; u < kVecPerLane; ++u) {
            update4<OPT>(sum[u], st[u], o);
#pragma unroll
            for (int i = 0; i < S; ++i) store_wm<RES>(stb[i], bo + u * 1024u, st[u][i]);
            if constexpr (PULL)
                for (int w = 0; w < n; ++w) store_out(ko[w] + offset, bo + u * 1024u, st[u][0]);
        }
    }
    for (uint32_t v = nfull + lane; v < nvec; v += 64u) {
        const uint32_t bo = v * 16u;
        const f4 s = sum_any(kp, n, offset, bo);
        f4 st[S];
#pragma unroll
        for (int i = 0; i < S; ++i) st[i] = load_wm<RES>(stb[i], bo);
        update4<OPT>(s, st, o);
#pragma unroll
        for (int i = 0; i < S; ++i) store_wm<RES>(stb[i], bo, st[i]);
        if constexpr (PULL)
            for (int w = 0; w < n; ++w) store_out(ko[w] + offset, bo, st[0]);
    }
    if (lane < rem) {
        const int64_t i = int64_t(nvec) * 4 + lane;
        float s = load1(kp[0] + offset, i);
        for (int w = 1; w < n; ++w) s = s + load1(kp[w] + offset, i);
        float st[S];
#pragma unroll
        for (int k = 0; k < S; ++k) st[k] = load1(stb[k], i);
        update<OPT>(s, st, o);
#pragma unroll
        for (int k = 0; k < S; ++k) store1(stb[k], i, st[k]);
        if constexpr (PULL)
            for (int w = 0; w < n; ++w) store1(ko[w] + offset, i, st[0]);
    }
}

// One bin of the any-N kernel: full tiles [tb, te), then remainders [rb, re).
template <int OPT, bool RES, bool PULL>
__device__ __forceinline__ void any_bin(const DevTile* __restrict__ tiles, int32_t tb, int32_t te,
                                        const DevRem* __restrict__ rems, int32_t rb, int32_t re,
                                        const float* const* __restrict__ grads,
                                        float* const* __restrict__ outs, float* const* state,
                                        int n, OptArgs o) {
    constexpr int S = kStates<OPT>;
    for (int32_t t = tb; t < te; ++t) {
        const DevTile tl = tiles[t];
        float* stb[S];
#pragma unroll
        for (int i = 0; i < S; ++i) stb[i] = state[i] + tl.arena_offset;
        run_any<OPT, RES, PULL>(grads + int64_t(tl.key) * n,
                                PULL ? outs + int64_t(tl.key) * n : nullptr, n,
                                int64_t(tl.vec) * 4, stb, uint32_t(kTileElems / 4), 0u, o);
    }
    for (int32_t r = rb; r < re; ++r) {
        const DevRem rm = rems[r];
        float* stb[S];
#pragma unroll
        for (int i = 0; i < S; ++i) stb[i] = state[i] + rm.arena_offset;
        run_any<OPT, RES, PULL>(grads + int64_t(rm.key) * n,
                                PULL ? outs + int64_t(rm.key) * n : nullptr, n, rm.offset, stb,
                                uint32_t(rm.count) >> 2, uint32_t(rm.count) & 3u, o);
    }
}

// (A launch built on the device has heads but no bin offsets, so the bins are
// read from the heads.)
template <int OPT, bool PULL>
__global__ __launch_bounds__(kBlockThreads) void fused_step_any(PHUB_KERNEL_ARGS) {
    float* const state[3] = {weights, moments, second};
    const uint32_t wave = wave_index();
    const WaveHead h = heads[wave];
    any_bin<OPT, false, PULL>(tiles, h.tiles_streamed[0], h.tiles_streamed[1], rems,
                              h.rems_streamed[0], h.rems_streamed[1], grads, outs, state,
                              num_workers, o);
    any_bin<OPT, true, PULL>(tiles, h.tiles_resident[0], h.tiles_resident[1], rems,
                             h.rems_resident[0], h.rems_resident[1], grads, outs, state,
                             num_workers, o);
}

// Ablation: the unfused ("wide") form of the step, kept to measure what
// fusion saves.  Pass 1 sums the N gradients of every element in worker
// order and writes the sum to a merge buffer laid out like W; pass 2 reads
// the merge buffer and the state and runs the optimizer.  Same arithmetic,
// same schedule, (N + 2 S + 2) * 4 bytes per element instead of
// (N + 2 S) * 4, and two launches.
__device__ __forceinline__ void aggregate_range(const float* const* kp, int n, int64_t offset,
                                                float* out, uint32_t nvec, uint32_t rem) {
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t v = lane; v < nvec; v += 64u)
        store_out(out, v * 16u, sum_any(kp, n, offset, v * 16u));
    if (lane < rem) {
        const int64_t i = int64_t(nvec) * 4 + lane;
        float s = load1(kp[0] + offset, i);
        for (int w = 1; w < n; ++w) s = s + load1(kp[w] + offset, i);
        store1(out, i, s);
    }
}

template <int OPT, bool RES>
__device__ __forceinline__ void optimize_range(const float* sum, float* const* stb, uint32_t nvec,
                                               uint32_t rem, OptArgs o) {
    constexpr int S = kStates<OPT>;
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t v = lane; v < nvec; v += 64u) {
        const uint32_t bo = v * 16u;
        const f4 s = load_stream(sum, bo);
        f4 st[S];
#pragma unroll
        for (int i = 0; i < S; ++i) st[i] = load_wm<RES>(stb[i], bo);
        update4<OPT>(s, st, o);
#pragma unroll
        for (int i = 0; i < S; ++i) store_wm<RES>(stb[i], bo, st[i]);
    }
    if (lane < rem) {
        const int64_t i = int64_t(nvec) * 4 + lane;
        float st[S];
#pragma unroll
        for (int k = 0; k < S; ++k) st[k] = load1(stb[k], i);
        update<OPT>(load1(sum, i), st, o);
#pragma unroll
        for (int k = 0; k < S; ++k) store1(stb[k], i, st[k]);
    }
}

__global__ __launch_bounds__(kBlockThreads) void aggregate_only(PHUB_KERNEL_ARGS, float* merge) {
    const uint32_t wave = wave_index();
    const uint32_t bins = gridDim.x * kWavesPerBlock;
    const int n = num_workers;
    for (uint32_t bin : {wave, bins + wave}) {
        for (int32_t t = tile_begin[bin]; t < tile_begin[bin + 1]; ++t) {
            const DevTile tl = tiles[t];
            aggregate_range(grads + int64_t(tl.key) * n, n, int64_t(tl.vec) * 4,
                            merge + tl.arena_offset, uint32_t(kTileElems / 4), 0u);
        }
        for (int32_t r = rem_begin[bin]; r < rem_begin[bin + 1]; ++r) {
            const DevRem rm = rems[r];
            aggregate_range(grads + int64_t(rm.key) * n, n, rm.offset, merge + rm.arena_offset,
                            uint32_t(rm.count) >> 2, uint32_t(rm.count) & 3u);
        }
    }
}

template <int OPT, bool RES>
__device__ __forceinline__ void optimize_bin(const DevTile* __restrict__ tiles, int32_t tb,
                                             int32_t te, const DevRem* __restrict__ rems,
                                             int32_t rb, int32_t re, const float* merge,
                                             float* const* state, OptArgs o) {
    constexpr int S = kStates<OPT>;
    for (int32_t t = tb; t < te; ++t) {
        const DevTile tl = tiles[t];
        float* stb[S];
#pragma unroll
        for (int i = 0; i < S; ++i) stb[i] = state[i] + tl.arena_offset;
        optimize_range<OPT, RES>(merge + tl.arena_offset, stb, uint32_t(kTileElems / 4), 0u, o);
    }
    for (int32_t r = rb; r < re; ++r) {
        const DevRem rm = rems[r];
        float* stb[S];
#pragma unroll
        for (int i = 0; i < S; ++i) stb[i] = state[i] + rm.arena_offset;
        optimize_range<OPT, RES>(merge + rm.arena_offset, stb, uint32_t(rm.count) >> 2,
                                 uint32_t(rm.count) & 3u, o);
    }
}

template <int OPT>
__global__ __launch_bounds__(kBlockThreads) void optimize_only(PHUB_KERNEL_ARGS, float* merge) {
    float* const state[3] = {weights, moments, second};
    const uint32_t wave = wave_index();
    const uint32_t bins = gridDim.x * kWavesPerBlock;
    optimize_bin<OPT, true>(tiles, tile_begin[wave], tile_begin[wave + 1], rems, rem_begin[wave],
                            rem_begin[wave + 1], merge, state, o);
    optimize_bin<OPT, false>(tiles, tile_begin[bins + wave], tile_begin[bins + wave + 1], rems,
                             rem_begin[bins + wave], rem_begin[bins + wave + 1], merge, state, o);
}

// -------------------------------------------------------------- launchers

#define PHUB_LAUNCH_ARGS                                                                     \
    p.tiles, p.tile_begin, p.rems, p.rem_begin, p.heads, p.grads, p.outs, p.weights,         \
        p.moments,                                                                           \
        p.second, p.opt, p.num_workers, p.pool, p.pool_count, p.pool_counters, p.pool_launch

template <int OPT, bool PULL>
hipError_t launch_any(const StepParams& p, int grid, hipStream_t stream) {
    if constexpr (!PULL) {
        const AnyKernel k = any_kernel(p.num_workers, p.load);
        if (k == kAnyStream) return launch_fused_step_many(p, OPT, grid, stream);
        if (k == kAnyStreamShared) return launch_fused_step_many_shared(p, OPT, grid, stream);
    }
    hipLaunchKernelGGL((fused_step_any<OPT, PULL>), dim3(grid), dim3(kBlockThreads), 0, stream,
                       PHUB_LAUNCH_ARGS);
    return hipGetLastError();
}

// (A load window that takes more than three phases, in a build that sets its
// depth, has no fixed-N kernel.)
template <int NW, int OPT, bool PULL>
hipError_t launch_one(const StepParams& p, int grid, hipStream_t stream) {
    constexpr int S = kStates<OPT>;
    if constexpr (kPhases<NW, S, true> <= 3 && kPhases<NW, S, false> <= 3) {
        hipLaunchKernelGGL((fused_step_fixed<NW, OPT, PULL>), dim3(grid), dim3(kBlockThreads), 0,
                           stream, PHUB_LAUNCH_ARGS);
        return hipGetLastError();
    } else {
        return launch_any<OPT, PULL>(p, grid, stream);
    }
}

template <int OPT, bool PULL>
hipError_t launch_pull(const StepParams& p, int grid, hipStream_t stream) {
    static_assert(kMaxFixedWorkers == 16, "one case per fixed worker count");
    static_assert(has_fixed_kernel(20) && has_fixed_kernel(24) && has_fixed_kernel(32),
                  "the larger counts below");
    if constexpr (!PULL)  // (the streamed walk takes no tile pool)
        if (p.pool_count == 0 &&
            takes_stream(p.num_workers, kStates<OPT>, p.load, int64_t(grid) * kWavesPerBlock))
            return launch_stream<OPT>(p, grid, stream);
    switch (p.num_workers) {
        case 1: return launch_one<1, OPT, PULL>(p, grid, stream);
        case 2: return launch_one<2, OPT, PULL>(p, grid, stream);
        case 3: return launch_one<3, OPT, PULL>(p, grid, stream);
        case 4: return launch_one<4, OPT, PULL>(p, grid, stream);
        case 5: return launch_one<5, OPT, PULL>(p, grid, stream);
        case 6: return launch_one<6, OPT, PULL>(p, grid, stream);
        case 7: return launch_one<7, OPT, PULL>(p, grid, stream);
        case 8: return launch_one<8, OPT, PULL>(p, grid, stream);
        case 9: return launch_one<9, OPT, PULL>(p, grid, stream);
        case 10: return launch_one<10, OPT, PULL>(p, grid, stream);
        case 11: return launch_one<11, OPT, PULL>(p, grid, stream);
        case 12: return launch_one<12, OPT, PULL>(p, grid, stream);
        case 13: return launch_one<13, OPT, PULL>(p, grid, stream);
        case 14: return launch_one<14, OPT, PULL>(p, grid, stream);
        case 15: return launch_one<15, OPT, PULL>(p, grid, stream);
        case 16: return launch_one<16, OPT, PULL>(p, grid, stream);
        case 20: return launch_one<20, OPT, PULL>(p, grid, stream);
        case 24: return launch_one<24, OPT, PULL>(p, grid, stream);
        case 32: return launch_one<32, OPT, PULL>(p, grid, stream);
        default: return launch_any<OPT, PULL>(p, grid, stream);
    }
}

template <int OPT>
hipError_t launch_unfused(const StepParams& p, int grid, hipStream_t stream) {
    hipLaunchKernelGGL(aggregate_only, dim3(grid), dim3(kBlockThreads), 0, stream,
                       PHUB_LAUNCH_ARGS, p.merge);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    hipLaunchKernelGGL((optimize_only<OPT>), dim3(grid), dim3(kBlockThreads), 0, stream,
                       PHUB_LAUNCH_ARGS, p.merge);
    return hipGetLastError();
}

}  // namespace

// The launchers of one optimizer, with (PULL) and without model buffers.
// Compiled on its own, this file holds all of them; the library's build
// compiles it once per launcher (PHUB_STEP_PART = 2 * optimizer + PULL) so
// that the parts compile side by side, the rest of the file in part 0.
template <int OPT, bool PULL>
hipError_t launch_step(const StepParams& p, int grid, hipStream_t stream);

#define PHUB_LAUNCH_STEP(OPT, PULL)                                                      \
    template <>                                                                          \
    hipError_t launch_step<OPT, PULL>(const StepParams& p, int grid, hipStream_t stream) { \
        if constexpr (!PULL)                                                             \
            if (p.merge) return launch_unfused<OPT>(p, grid, stream);                    \
        return launch_pull<OPT, PULL>(p, grid, stream);                                  \
    }
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 0
PHUB_LAUNCH_STEP(kOptMomentum, false)
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 1
PHUB_LAUNCH_STEP(kOptMomentum, true)
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 2
PHUB_LAUNCH_STEP(kOptNesterov, false)
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 3
PHUB_LAUNCH_STEP(kOptNesterov, true)
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 4
PHUB_LAUNCH_STEP(kOptSgd, false)
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 5
PHUB_LAUNCH_STEP(kOptSgd, true)
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 6
PHUB_LAUNCH_STEP(kOptAdam, false)
#endif
#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 7
PHUB_LAUNCH_STEP(kOptAdam, true)
#endif

#if !defined(PHUB_STEP_PART) || PHUB_STEP_PART == 0
namespace {

template <int NW, int S>
constexpr bool fixed_launchable() {
    return kPhases<NW, S, true> <= 3 && kPhases<NW, S, false> <= 3;
}

template <int S>
bool fixed_launchable_n(int n) {
    switch (n) {
        case 1: return fixed_launchable<1, S>();
        case 2: return fixed_launchable<2, S>();
        case 3: return fixed_launchable<3, S>();
        case 4: return fixed_launchable<4, S>();
        case 5: return fixed_launchable<5, S>();
        case 6: return fixed_launchable<6, S>();
        case 7: return fixed_launchable<7, S>();
        case 8: return fixed_launchable<8, S>();
        case 9: return fixed_launchable<9, S>();
        case 10: return fixed_launchable<10, S>();
        case 11: return fixed_launchable<11, S>();
        case 12: return fixed_launchable<12, S>();
        case 13: return fixed_launchable<13, S>();
        case 14: return fixed_launchable<14, S>();
        case 15: return fixed_launchable<15, S>();
        case 16: return fixed_launchable<16, S>();
        case 20: return fixed_launchable<20, S>();
        case 24: return fixed_launchable<24, S>();
        case 32: return fixed_launchable<32, S>();
        default: return false;
    }
}

}  // namespace

bool takes_tile_pool(int num_workers, int optimizer) {
    switch (optimizer) {
        case kOptMomentum:
        case kOptNesterov: return fixed_launchable_n<2>(num_workers);
        case kOptSgd: return fixed_launchable_n<1>(num_workers);
        case kOptAdam: return fixed_launchable_n<3>(num_workers);
        default: return false;
    }
}

hipError_t launch_fused_step(const StepParams& p, int optimizer, int grid, hipStream_t stream) {
    if (p.pool_count > 0 && (p.merge || !takes_tile_pool(p.num_workers, optimizer)))
        return hipErrorInvalidValue;  // only the fixed-N fused kernels walk a pool
    if (!p.merge && !p.heads) return hipErrorInvalidValue;  // the fused kernels read them
    const bool pull = p.outs && !p.merge;
    switch (optimizer) {
        case kOptMomentum:
            return pull ? launch_step<kOptMomentum, true>(p, grid, stream)
                        : launch_step<kOptMomentum, false>(p, grid, stream);
        case kOptNesterov:
            return pull ? launch_step<kOptNesterov, true>(p, grid, stream)
                        : launch_step<kOptNesterov, false>(p, grid, stream);
        case kOptSgd:
            return pull ? launch_step<kOptSgd, true>(p, grid, stream)
                        : launch_step<kOptSgd, false>(p, grid, stream);
        case kOptAdam:
            return pull ? launch_step<kOptAdam, true>(p, grid, stream)
                        : launch_step<kOptAdam, false>(p, grid, stream);
        default: return hipErrorInvalidValue;
    }
}

#endif  // PHUB_STEP_PART

}  // namespace phub
