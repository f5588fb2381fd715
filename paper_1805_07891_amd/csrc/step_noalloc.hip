// One exchange step that allocates nothing: phub_step_noalloc.
//
// For callers that cannot allocate device memory (serving loops that must
// not call hipMalloc, harnesses that forbid allocation).  The caller passes
// the gradients and the master weights and momentum; everything else the
// fused kernel reads (the chunk schedule of section 3.2.4 in its device form
// and the gradient pointer table) goes into `scratch` below, and the key
// entries it is built from into `key_entries`: file-scope device arrays that
// each GPU holds for the life of the process (4 and 2.7 MiB).  The kernel
// is the job path's fused kernel, so the results are those of phub_init +
// phub_push_all + phub_step on the same inputs (they do not depend on the
// schedule).
//
// A call has no earlier schedule to reuse, so the schedule is built on the
// device: the host sends one 16-byte entry per key and the pointer table,
// and one small kernel writes the tile and remainder descriptors and the
// wave heads, every descriptor's place in closed form (tiles dealt to the
// waves in turn, which is what the longest-processing-time-first rule does
// with equal items; then the remainders).  The words travel as kernel
// arguments, so the call neither waits for the stream nor reads host memory
// after it returns.  Measured (MI355X, 161 keys, 25.6 M parameters, 8
// workers, a call): schedule built on the host, copied and waited for 1976
// us, this 201 us, of which the step's kernel takes 190.
//
// An array's name in host code is a host-side stand-in, not a device address:
// its device address is taken once per device with hipGetSymbolAddress, with
// that device current, and only that address is used from host code.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "kernels.hpp"
#include "phub.h"
#include "plan.hpp"

// Largest schedule plus pointer table one call can hold: 4 MiB, enough for
// about 240 M parameters in 1024-element tiles (16 bytes each, beside the
// 128 KB of wave heads) with the
// pointer table of thousands of (worker, key) pairs.
#define PHUB_NOALLOC_SCRATCH_BYTES (size_t(4) << 20)

static __device__ __align__(256) unsigned char scratch[PHUB_NOALLOC_SCRATCH_BYTES];

// The key entries of a call: a key with elements takes a remainder or tiles
// of the scratch array and a row of its pointer table, so this many keys
// cannot be exceeded.
#define PHUB_NOALLOC_MAX_KEYS (PHUB_NOALLOC_SCRATCH_BYTES / 24)

namespace {

constexpr size_t kScratchBytes = PHUB_NOALLOC_SCRATCH_BYTES;

// One key with elements, in key order; the prefix sums place its tiles and
// its remainder.
struct KeyEntry {
    uint32_t arena64;     // first element in the arenas / 64
    uint32_t tile_begin;  // full tiles of the keys before it
    uint32_t rem_begin;   // remainders of the keys before it
    uint32_t rem_count;   // elements of its own remainder (0: none)
};
static_assert(sizeof(KeyEntry) == 16, "KeyEntry layout");
static __device__ __align__(256) KeyEntry key_entries[PHUB_NOALLOC_MAX_KEYS];

// Words sent to the device as the arguments of one launch.
constexpr int kPutWords = 480;
struct PutArgs {
    uint64_t w[kPutWords];
};
// Above this many launches the words are copied instead, with a wait for the
// stream.  Measured with steps of a few microseconds (host time of a call,
// launches against copies): 15 against 26 us at one launch, 33 against 36 at
// 4, 53 against 59 at 7, 99 against 76 at 14, 184 against 117 at 27; with
// longer steps the launches stay hidden behind the step before, and the
// wait does not.
constexpr size_t kMaxPutLaunches = 16;

// dst_a[0, n_a) and dst_b[0, n_b) from the arguments' first n_a + n_b words.
__global__ __launch_bounds__(kPutWords) void put_words(PutArgs a, uint64_t* __restrict__ dst_a, int n_a,
                                                       uint64_t* __restrict__ dst_b, int n_b) {
    const int i = int(threadIdx.x);
    if (i < n_a)
        dst_a[i] = a.w[i];
    else if (i < n_a + n_b)
        dst_b[i - n_a] = a.w[i];
}

// Position of bin b's first entry when `count` entries are dealt to `bins`
// bins in turn and listed bin by bin, and how many it has.
__host__ __device__ inline uint32_t dealt_begin(uint32_t count, uint32_t bins, uint32_t b) {
    const uint32_t extra = count % bins;
    return b * (count / bins) + (b < extra ? b : extra);
}
__host__ __device__ inline uint32_t dealt_count(uint32_t count, uint32_t bins, uint32_t b) {
    return count / bins + (b < count % bins ? 1u : 0u);
}

// Last key whose prefix sum is <= i: the key that holds tile (or remainder)
// i, since the keys without one share the sum of the next that has.
template <bool REM>
__device__ inline uint32_t find_key(const KeyEntry* keys, uint32_t num_keys, uint32_t i) {
    uint32_t lo = 0, hi = num_keys;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if ((REM ? keys[mid].rem_begin : keys[mid].tile_begin) <= i)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

__device__ inline phub::DevTile tile_desc(const KeyEntry* keys, uint32_t num_keys, uint32_t i) {
    const uint32_t k = find_key<false>(keys, num_keys, i);
    const uint32_t t = i - keys[k].tile_begin;  // the key's t-th tile
    return {int64_t(keys[k].arena64) * 64 + int64_t(t) * phub::kTileElems, int32_t(k),
            t * uint32_t(phub::kTileElems / 4)};
}

__device__ inline phub::DevRem rem_desc(const KeyEntry* keys, uint32_t num_keys, uint32_t num_tiles,
                                        uint32_t k) {
    const uint32_t end = k + 1 < num_keys ? keys[k + 1].tile_begin : num_tiles;
    const int64_t done = int64_t(end - keys[k].tile_begin) * phub::kTileElems;
    return {int64_t(keys[k].arena64) * 64 + done, done, int32_t(k), int32_t(keys[k].rem_count), 0};
}

// The schedule of a launch of `bins` waves: thread i writes tile i, key i's
// remainder and wave i's head.  Tile i goes to wave i mod bins; remainder r
// to wave (num_tiles + r) mod bins, so that the waves with one tile less
// come first.  About 1 us: bound by the search's dependent loads, which the
// keys' copy in LDS shortens.
constexpr uint32_t kLdsKeys = 2048;
__global__ __launch_bounds__(256) void build_schedule(const KeyEntry* __restrict__ entries,
                                                      uint32_t num_keys, uint32_t num_tiles,
                                                      uint32_t num_rems, uint32_t bins,
                                                      phub::DevTile* __restrict__ tiles,
                                                      phub::DevRem* __restrict__ rems,
                                                      phub::WaveHead* __restrict__ heads) {
    __shared__ KeyEntry lds[kLdsKeys];
    const KeyEntry* keys = entries;
    if (num_keys <= kLdsKeys) {
        for (uint32_t k = threadIdx.x; k < num_keys; k += blockDim.x) lds[k] = entries[k];
        __syncthreads();
        keys = lds;
    }
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < num_tiles)
        tiles[dealt_begin(num_tiles, bins, i % bins) + i / bins] = tile_desc(keys, num_keys, i);
    if (i < num_keys && keys[i].rem_count) {
        const uint32_t r = keys[i].rem_begin;
        rems[dealt_begin(num_rems, bins, r % bins) + r / bins] =
            rem_desc(keys, num_keys, num_tiles, i);
    }
    if (i < bins) {
        phub::WaveHead h{};
        const uint32_t t0 = dealt_begin(num_tiles, bins, i), nt = dealt_count(num_tiles, bins, i);
        h.tiles_streamed[0] = int32_t(t0);
        h.tiles_streamed[1] = int32_t(t0 + nt);
        if (nt) h.first_streamed = tile_desc(keys, num_keys, i);
        const uint32_t r = (i + bins - num_tiles % bins) % bins;  // its first remainder
        const uint32_t r0 = dealt_begin(num_rems, bins, r), nr = dealt_count(num_rems, bins, r);
        h.rems_streamed[0] = int32_t(r0);
        h.rems_streamed[1] = int32_t(r0 + nr);
        if (nr) {
            const uint32_t k = find_key<true>(keys, num_keys, r);
            h.first_rem_streamed = rem_desc(keys, num_keys, num_tiles, k);
        }
        heads[i] = h;
    }
}
constexpr int64_t kArenaAlign = 64;  // elements: key slices of the arena start 256-byte aligned
constexpr size_t kRegionAlign = 256;

// What one device needs for a call, found once per device.
struct DeviceSetup {
    unsigned char* scratch = nullptr;  // device address of `scratch` on this device
    KeyEntry* keys = nullptr;          // and of `key_entries`
    int compute_units = 0;
    int64_t wall_clock_khz = 0;
};

std::mutex g_setup_mu;
std::unordered_map<int, DeviceSetup> g_setup;

// The device's setup, found on the first call made on it (the device is
// current during the call).
int device_setup(int device, DeviceSetup* out) {
    std::lock_guard<std::mutex> lk(g_setup_mu);
    auto it = g_setup.find(device);
    if (it != g_setup.end()) {
        *out = it->second;
        return PHUB_OK;
    }
    DeviceSetup s;
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
        return phub::report_error(PHUB_EHIP, std::string("hipGetSymbolAddress(scratch) failed: ") +
                                                 hipGetErrorString(e));
    s.scratch = static_cast<unsigned char*>(ptr);
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(key_entries));
    if (e != hipSuccess || !ptr)
        return phub::report_error(PHUB_EHIP, std::string("hipGetSymbolAddress(key_entries) failed: ") +
                                                 hipGetErrorString(e));
    s.keys = static_cast<KeyEntry*>(ptr);
    e = hipDeviceGetAttribute(&s.compute_units, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess || s.compute_units < 1)
        return phub::report_error(PHUB_EHIP, "hipDeviceGetAttribute(CU count) failed");
    int khz = 0;
    e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device);
    if (e != hipSuccess || khz < 1)
        return phub::report_error(PHUB_EHIP, "hipDeviceGetAttribute(wall clock rate) failed");
    s.wall_clock_khz = khz;
    g_setup[device] = s;
    *out = s;
    return PHUB_OK;
}

size_t align_up(size_t x) { return (x + kRegionAlign - 1) / kRegionAlign * kRegionAlign; }

std::string fmt(const char* f, long long a, long long b = 0, long long c = 0) {
    char buf[256];
    std::snprintf(buf, sizeof buf, f, a, b, c);
    return buf;
}

}  // namespace

extern "C" int phub_step_noalloc(int num_workers, int num_keys, const int64_t* key_elems,
                                 int64_t chunk_bytes, float lr, float momentum,
                                 float weight_decay, int nesterov, const float* const* grads,
                                 float* weights, float* moments, void* hip_stream) {
    using phub::report_error;
    {
        const std::string err = phub::validate_shape(num_workers, num_keys, key_elems, chunk_bytes);
        if (!err.empty()) return report_error(PHUB_EINVAL, err);
    }
    if (!std::isfinite(lr) || !std::isfinite(momentum) || !std::isfinite(weight_decay))
        return report_error(PHUB_EINVAL, "lr, momentum and weight_decay must be finite");
    if (!grads) return report_error(PHUB_EINVAL, "grads is NULL");
    // the arena layout of a job's state: key slices padded to 64 elements
    std::vector<int64_t> arena_offset;
    try {
        arena_offset.resize(num_keys);
    } catch (const std::bad_alloc&) {
        return report_error(PHUB_ENOMEM, "host allocation of the key offsets failed");
    }
    int64_t arena_elems = 0;
    for (int k = 0; k < num_keys; ++k) {
        if (key_elems[k] >= phub::kMaxDeviceKeyElems)
            return report_error(PHUB_EINVAL, fmt("key_elems[%lld] = %lld exceeds the %lld elements a key may hold",
                                                 k, key_elems[k], phub::kMaxDeviceKeyElems - 1));
        arena_offset[k] = arena_elems;
        arena_elems += (key_elems[k] + kArenaAlign - 1) / kArenaAlign * kArenaAlign;
    }
    if (arena_elems > 0) {
        if (!weights || !moments) return report_error(PHUB_EINVAL, "weights or moments is NULL");
        if (reinterpret_cast<uintptr_t>(weights) % 16 || reinterpret_cast<uintptr_t>(moments) % 16)
            return report_error(PHUB_EINVAL, "weights and moments must be 16-byte aligned");
    }
    for (int w = 0; w < num_workers; ++w)
        for (int k = 0; k < num_keys; ++k) {
            const float* g = grads[size_t(w) * num_keys + k];
            if (!g && key_elems[k] != 0)
                return report_error(PHUB_EINVAL, fmt("gradient of worker %lld for key %lld is NULL", w, k));
            if (reinterpret_cast<uintptr_t>(g) % 16)
                return report_error(PHUB_EINVAL,
                                    fmt("gradient of worker %lld for key %lld is not 16-byte aligned", w, k));
        }
    // Bound the scratch need before any HIP call: the schedule holds at most
    // one tile per 1024 elements plus a remainder per segment, and a bin
    // table; the pointer table one pointer per (worker, key).  The exact
    // size is checked again once the schedule is built.
    const size_t table_bytes = size_t(num_workers) * size_t(num_keys) * sizeof(const float*);
    if (table_bytes > kScratchBytes || arena_elems / phub::kTileElems * int64_t(sizeof(phub::DevTile)) >
                                           int64_t(kScratchBytes))
        return report_error(PHUB_EINVAL,
                            fmt("the step needs more than the %lld bytes of scratch this entry point "
                                "has (%lld parameters, %lld gradient pointers)",
                                (long long)kScratchBytes, arena_elems,
                                (long long)num_workers * num_keys));

    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return report_error(PHUB_EHIP, "hipGetDevice failed");
    DeviceSetup setup;
    if (int rc = device_setup(device, &setup)) return rc;

    const int grid = setup.compute_units;
    const int bins = grid * (phub::kBlockThreads / 64);
    // Scratch layout, each region 256-byte aligned: the waves' heads, tiles,
    // remainders, gradient pointer table (a row per key with elements).  The
    // limit is the one of the schedule cut at chunk_bytes (which needs at
    // least as much), with its two tables of 2 * bins + 1 bin offsets.
    const phub::LptCounts lpt =
        phub::lpt_counts(num_keys, key_elems, chunk_bytes, 128 * bins, phub::kTileElems);
    if (lpt.tiles == 0 && lpt.rems == 0) return PHUB_OK;  // every key is empty
    const size_t head_bytes = align_up(size_t(bins) * sizeof(phub::WaveHead));
    const size_t total = 2 * align_up((2 * size_t(bins) + 1) * sizeof(int32_t)) + head_bytes +
                         align_up(size_t(lpt.tiles) * sizeof(phub::DevTile)) +
                         align_up(size_t(lpt.rems) * sizeof(phub::DevRem)) + table_bytes;
    if (total > kScratchBytes)
        return report_error(PHUB_EINVAL,
                            fmt("the step needs %lld bytes of scratch; this entry point has %lld",
                                (long long)total, (long long)kScratchBytes));
    std::vector<KeyEntry> keys;
    std::vector<uint64_t> words;  // the pointer table [row * num_workers + worker], the entries
    uint32_t num_tiles = 0, num_rems = 0;
    try {
        keys.reserve(num_keys);
        words.reserve(size_t(num_workers) * num_keys + 2 * size_t(num_keys));
        for (int k = 0; k < num_keys; ++k) {
            if (key_elems[k] == 0) continue;
            const uint32_t rem = uint32_t(key_elems[k] % phub::kTileElems);
            keys.push_back({uint32_t(arena_offset[k] / kArenaAlign), num_tiles, num_rems, rem});
            num_tiles += uint32_t(key_elems[k] / phub::kTileElems);
            num_rems += rem ? 1 : 0;
            for (int w = 0; w < num_workers; ++w)
                words.push_back(reinterpret_cast<uint64_t>(grads[size_t(w) * num_keys + k]));
        }
        const size_t n = words.size();
        words.resize(n + 2 * keys.size());
        std::memcpy(words.data() + n, keys.data(), keys.size() * sizeof(KeyEntry));
    } catch (const std::bad_alloc&) {
        return report_error(PHUB_ENOMEM, "host allocation of the key table failed");
    }
    const size_t num_entries = keys.size();
    const size_t off_tiles = head_bytes;
    const size_t off_rems = align_up(off_tiles + num_tiles * sizeof(phub::DevTile));
    const size_t off_grads = align_up(off_rems + num_rems * sizeof(phub::DevRem));
    const size_t num_ptrs = words.size() - 2 * num_entries;
    if (off_grads + num_ptrs * sizeof(uint64_t) > kScratchBytes || num_entries > PHUB_NOALLOC_MAX_KEYS)
        return report_error(PHUB_EINVAL, "schedule too large");

    // Everything below follows the stream's earlier work (an earlier call's
    // kernel may still read the scratch).  A captured call would replay with
    // these pointers into an array that other calls write: refused.
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    e = hipStreamIsCapturing(stream, &capture);
    if (e != hipSuccess || capture != hipStreamCaptureStatusNone)
        return report_error(PHUB_EHIP, "phub_step_noalloc on a stream that is being captured");
    uint64_t* const d_ptrs = reinterpret_cast<uint64_t*>(setup.scratch + off_grads);
    uint64_t* const d_keys = reinterpret_cast<uint64_t*>(setup.keys);
    if (words.size() <= kMaxPutLaunches * kPutWords) {
        for (size_t at = 0; at < words.size(); at += kPutWords) {
            PutArgs a;
            const size_t n = std::min<size_t>(kPutWords, words.size() - at);
            std::memcpy(a.w, words.data() + at, n * sizeof(uint64_t));
            // words [at, at + n) up to num_ptrs are pointers, the rest entries
            const size_t na = at < num_ptrs ? std::min(n, num_ptrs - at) : 0;
            hipLaunchKernelGGL(put_words, dim3(1), dim3(kPutWords), 0, stream, a,
                               d_ptrs + (na ? at : 0), int(na),
                               d_keys + (n > na ? at + na - num_ptrs : 0), int(n - na));
            e = hipGetLastError();
            if (e != hipSuccess)
                return report_error(PHUB_EHIP, std::string("launch of the upload kernel failed: ") +
                                                   hipGetErrorString(e));
        }
    } else {
        // two copies, then a wait, so that the host image may go
        e = hipMemcpyAsync(d_ptrs, words.data(), num_ptrs * sizeof(uint64_t), hipMemcpyHostToDevice,
                           stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(d_keys, words.data() + num_ptrs, num_entries * sizeof(KeyEntry),
                               hipMemcpyHostToDevice, stream);
        if (e != hipSuccess)
            return report_error(PHUB_EHIP, std::string("hipMemcpyAsync (scratch) failed: ") +
                                               hipGetErrorString(e));
        e = hipStreamSynchronize(stream);
        if (e != hipSuccess)
            return report_error(PHUB_EHIP, std::string("hipStreamSynchronize failed: ") +
                                               hipGetErrorString(e));
    }
    phub::DevTile* const d_tiles = reinterpret_cast<phub::DevTile*>(setup.scratch + off_tiles);
    phub::DevRem* const d_rems = reinterpret_cast<phub::DevRem*>(setup.scratch + off_rems);
    phub::WaveHead* const d_heads = reinterpret_cast<phub::WaveHead*>(setup.scratch);
    const uint32_t threads = std::max({num_tiles, uint32_t(num_entries), uint32_t(bins)});
    hipLaunchKernelGGL(build_schedule, dim3((threads + 255) / 256), dim3(256), 0, stream, setup.keys,
                       uint32_t(num_entries), num_tiles, num_rems, uint32_t(bins), d_tiles, d_rems,
                       d_heads);
    e = hipGetLastError();
    if (e != hipSuccess)
        return report_error(PHUB_EHIP, std::string("launch of the schedule kernel failed: ") +
                                           hipGetErrorString(e));

    phub::StepParams p{};
    p.heads = d_heads;
    p.load = {num_tiles, 0, num_rems, (int64_t(num_tiles) + bins - 1) / bins, bins};
    p.tiles = d_tiles;
    p.rems = d_rems;
    p.grads = reinterpret_cast<const float* const*>(d_ptrs);
    p.outs = nullptr;
    p.merge = nullptr;
    p.weights = weights;
    p.moments = moments;
    p.second = nullptr;
    p.opt.nlr = -lr;
    p.opt.mu = momentum;
    p.opt.wd = weight_decay;
    phub::write_phase_ticks(num_workers, 2, setup.wall_clock_khz, &p.opt.wb_period, &p.opt.wb_window);
    p.num_workers = num_workers;
    e = phub::launch_fused_step(p, nesterov ? phub::kOptNesterov : phub::kOptMomentum, grid, stream);
    if (e != hipSuccess)
        return report_error(PHUB_EHIP, std::string("launch of the fused step kernel failed: ") +
                                           hipGetErrorString(e));
    return PHUB_OK;
}
