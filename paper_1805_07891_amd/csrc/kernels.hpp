// Device-side data of the exchange step and its launcher.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "plan.hpp"

namespace phub {

#ifndef PHUB_BLOCK_THREADS
#define PHUB_BLOCK_THREADS 256
#endif

// Threads per workgroup; the kernels are compiled for exactly this size so
// that the register budget per lane follows from it.
constexpr int kBlockThreads = PHUB_BLOCK_THREADS;
static_assert(kBlockThreads >= 64 && kBlockThreads <= 1024 && kBlockThreads % 64 == 0,
              "block size must be a multiple of the wave size");

// A tile is what one wave moves per iteration of its hot loop: 4 float4 per
// lane of each array, i.e. 1024 elements (4 KB) of every gradient, of W and
// of M.
constexpr int kVecPerLane = 4;
constexpr int64_t kTileElems = 64 * 4 * kVecPerLane;

// Largest key the device descriptors address: a tile's float4 index is 32
// bits.
constexpr int64_t kMaxDeviceKeyElems = int64_t(1) << 34;

// One full tile (16 bytes): kTileElems elements of a key starting at
// element 4 * vec (keys therefore hold fewer than kMaxDeviceKeyElems).
struct DevTile {
    int64_t arena_offset;  // index of the tile's first element in the W and M arenas
    int32_t key;           // the key's row in the gradient pointer table
    uint32_t vec;          // index of the tile's first float4 within the key
};
static_assert(sizeof(DevTile) == 16, "DevTile layout");

// The rest of a segment after its full tiles (32 bytes): fewer than
// kTileElems elements, possibly with a ragged end of up to 3 elements.
struct DevRem {
    int64_t arena_offset;  // index of the first element in the W and M arenas
    int64_t offset;        // index of the first element within the key (multiple of 4)
    int32_t key;           // the key's row in the gradient pointer table
    int32_t count;         // elements, 1 .. kTileElems - 1
    int64_t pad;
};
static_assert(sizeof(DevRem) == 32, "DevRem layout");

// The start of one wave's work in a launch of the fused kernels (128
// bytes), read with one burst of scalar loads at the start of the launch:
// the wave's four bins (as offsets into the tile and remainder tables) and
// the first descriptor of each (zeros where the bin is empty).  Without it
// the first data load of a wave waits for the bin offsets, then for the
// first descriptor, then for the descriptor's pointer row; with it, only
// for the pointer row (one trip to memory less; about 0.4 us of a small
// job's launch on MI355X).
struct WaveHead {
    int32_t tiles_resident[2];   // [begin, end) into the tile table
    int32_t tiles_streamed[2];
    int32_t rems_resident[2];    // [begin, end) into the remainder table
    int32_t rems_streamed[2];
    DevTile first_resident;
    DevTile first_streamed;
    DevRem first_rem_resident;
    DevRem first_rem_streamed;
};
static_assert(sizeof(WaveHead) == 128, "WaveHead layout");

// Optimizers of the fused pass (pluggable, paper section 3.2.2).
enum OptKind : int {
    kOptMomentum = 0,  // SGD with momentum (state W, M)
    kOptNesterov = 1,  // SGD with Nesterov momentum (state W, M)
    kOptSgd = 2,       // plain SGD (state W)
    kOptAdam = 3,      // Adam with bias correction (state W, M, V)
};

// Worker counts 1 .. kMaxFixedWorkers, and 20, 24 and 32, have a
// compile-time kernel each; other counts take the any-N kernel.
constexpr int kMaxFixedWorkers = 16;

constexpr bool has_fixed_kernel(int num_workers) {
    return (num_workers >= 1 && num_workers <= kMaxFixedWorkers) || num_workers == 20 ||
           num_workers == 24 || num_workers == 32;
}

// Whether the window over a tile of a fixed-N fused pass (without pushpull)
// writes the streamed bin's state back in bursts through LDS, in the
// chip-wide write phases below (the stream walk always does: with Adam from
// 7 workers, kStreamBlock): from 6 workers for momentum and plain SGD, from
// 14 for Adam (measured on MI355X with nothing cached, against piece-by-piece
// write-back: momentum with 6-16 workers +0.7 to +4.5 points, plain SGD with
// 6-16 up to +0.8, Adam with 14 and 16 +2.7 and +1.7; with fewer workers 1.5
// to 15 points slower).  num_states: 1 plain SGD, 2 momentum, 3 Adam.
constexpr int kBurstMinWorkers[3] = {6, 6, 14};

constexpr bool burst_write_back(int num_workers, int num_states) {
    return has_fixed_kernel(num_workers) && num_states >= 1 && num_states <= 3 &&
           num_workers >= kBurstMinWorkers[num_states - 1];
}

// The burst write-back's stash: LDS per wave (the compute unit's 160 KB
// over its four waves), and how many tiles of state it holds for a job
// with num_states state arrays (a tile is 4 KB per array and wave).
constexpr int kStashBytesPerWave = 40 * 1024;
constexpr int stash_tiles(int num_states) {
    return num_states >= 1 ? kStashBytesPerWave / (num_states * 4 * 1024) : 0;
}

// Chip-wide write phases of the burst write-back.  Every wave of every
// launch reads the same constant-rate wall clock; the clock's time is cut
// into periods, and the first part of each period (the write window) is
// when waves write back their stashed state.  A period is about as many
// tiles of a wave's reads as the stash holds besides the tile in progress
// (4 of momentum's 5, 9 of plain SGD's 10, 2 of Adam's 3), at
// kWritePeriodNsPerStreamTile per element stream of a tile (N + 2 S
// streams: gradients, state read, state written) and stashed tile; the
// window is about one tile (kWriteWindowNs).  The host converts both to
// clock ticks.  By state arrays (plain SGD, momentum, Adam), so that a
// period is about 0.93 of the time a wave takes to fill its stash.  Swept
// on MI355X: momentum at 8 and 16 workers, 550-700 ns per stream and tile
// and 6-10 us windows lie within a point of each other, 800 ns with a 15.4
// us window 1-2.6 points below; plain SGD, 650 -> 600 ns at 6 to 64 workers
// +0.3 to +0.9 points (8 over 61.1 M parameters 0.834 -> 0.841); Adam, 650
// ns and 8 us -> 800 and 7 at 7 to 64 workers +0.1 to +1.7 points (8 over
// 61.1 M 0.809 -> 0.819).
constexpr int64_t kWritePeriodNsPerStreamTile[3] = {600, 650, 800};
constexpr int64_t kWriteWindowNs[3] = {8000, 8000, 7000};

// Write-phase period and window of the burst write-back in ticks of a wall
// clock running at clock_khz, for a job with num_workers gradients and
// num_states state arrays.
inline void write_phase_ticks(int num_workers, int num_states, int64_t clock_khz,
                              uint32_t* period, uint32_t* window) {
    const int64_t streams = num_workers + 2 * int64_t(num_states);
    const int64_t tiles = std::max<int64_t>(stash_tiles(num_states) - 1, 1);
    const int64_t p = kWritePeriodNsPerStreamTile[num_states - 1] * streams * tiles * clock_khz / 1000000;
    const int64_t w = kWriteWindowNs[num_states - 1] * clock_khz / 1000000;
    *period = uint32_t(std::min<int64_t>(std::max<int64_t>(p, 2), INT32_MAX));
    *window = uint32_t(std::min<int64_t>(std::max<int64_t>(w, 1), *period - 1));
}

// Counters of the dynamic schedule.  The waves of workgroup g take from
// counter g mod C (C = the launch's counters: kMaxPoolCounters, or fewer
// for a grid of fewer workgroups; one per XCD of MI355X, whose workgroups
// go to the XCDs in turn), counter c serving pool tiles c, c + C, c + 2 C,
// ...  Each readiness group has its own counters, each on its own 256-byte
// line, never reset: every launch of the group adds the same amount to
// counter c (the tiles it serves plus the waves that take from it, each
// wave taking once past its tiles), so the counter's value at the start of
// the group's launch number L (from 0) is L times that amount.
constexpr int kMaxPoolCounters = 8;
constexpr int kPoolCounterStride = 32;  // unsigned long long: 256 bytes

// Counters a launch of `grid` workgroups uses.
constexpr int pool_counter_count(int64_t grid) {
    return grid < kMaxPoolCounters ? int(grid) : kMaxPoolCounters;
}

// Tiles of a pool of `count` tiles that counter c of C serves.
constexpr int64_t pool_counter_tiles(int64_t count, int c, int counters) {
    return count > c ? (count - c + counters - 1) / counters : 0;
}

// Workgroups of a grid of `grid` that take from counter c of C.
constexpr int64_t pool_counter_groups(int64_t grid, int c, int counters) {
    return grid > c ? (grid - c + counters - 1) / counters : 0;
}

// Scalars of one launch.  For Adam, c1 = 1 - b1, c2 = 1 - b2 and the
// step's bias corrections k1 = lr / (1 - b1^t), k2 = 1 / (1 - b2^t) are
// computed on the host in double and rounded to fp32 once.
struct OptArgs {
    float nlr;  // -lr
    float mu;
    float wd;
    float b1, b2, c1, c2, k1, k2, eps;
    // burst write-back (see kWritePeriodNsPerStreamTile): the write phases'
    // period and window in ticks of the device's wall clock
    uint32_t wb_period;
    uint32_t wb_window;
};

// How a launch's full tiles lie on its waves.
struct TileLoad {
    int64_t streamed;  // full tiles of all streamed bins
    int64_t resident;  // full tiles of all cache-resident bins
    int64_t rems;      // remainders of all bins
    int64_t busiest;   // the most full tiles one wave has, of both
    int64_t waves;     // the launch's, at most one per SIMD of the device
};

// The schedule of one launch has two bins per wave.  With
// bins = grid * kBlockThreads / 64 waves, the bin tables hold 2 * bins + 1
// offsets: wave w's cache-resident bin is [begin[w], begin[w+1]) (its state
// stays in the memory-side cache between steps: cache-allocating loads and
// stores), its streamed bin [begin[bins+w], begin[bins+w+1]) (state read
// and written non-temporally).  The fused kernels walk the streamed bin
// first.
struct StepParams {
    const DevTile* tiles;         // grouped by bin
    const int32_t* tile_begin;    // 2 * bins + 1 offsets into tiles
    const DevRem* rems;           // grouped by bin
    const int32_t* rem_begin;     // 2 * bins + 1 offsets into rems
    const WaveHead* heads;        // one per wave (the fused kernels read these, not the offsets)
    TileLoad load;
    const float* const* grads;    // [row * num_workers + worker], 16-byte aligned
    float* const* outs;           // same layout: model buffers that receive w' (pushpull), or null
    float* merge;                 // unfused ablation: sum buffer laid out like W, or null (fused)
    float* weights;               // W arena
    float* moments;               // M arena (momentum, Adam's first moment), or null
    float* second;                // V arena (Adam's second moment), or null
    OptArgs opt;
    int num_workers;
    // dynamic schedule: the launch's streamed full tiles as one pool (the
    // streamed bins then hold only remainders), taken by the waves through
    // pool counters (see PoolCounters).  pool_count 0: none.
    const DevTile* pool;
    int32_t pool_count;
    unsigned long long* pool_counters;  // the group's counters, kPoolCounterStride apart
    uint64_t pool_launch;               // the group's launches before this one
};

// Whether the fused kernel for num_workers and optimizer (an OptKind) can
// walk a tile pool (the fixed-N kernels; not the any-N kernel).
bool takes_tile_pool(int num_workers, int optimizer);

// A part of a key scheduled on its own (a job's cache-resident or
// streamed part of the key): the key's row in the gradient pointer table,
// the part's first element within the key (a multiple of 4) and its
// element count.
struct VirtualKey {
    int row;
    int64_t base;
    int64_t elems;
};

// Device form of schedules: full tiles and remainders grouped by bin, and
// offsets into them (each bin ends where the next begins).
struct DeviceTables {
    std::vector<DevTile> tiles;
    std::vector<DevRem> rems;
    std::vector<int32_t> tile_begin;
    std::vector<int32_t> rem_begin;
};

// Appends the device form of `plan` (built over `vkeys`) to `out`: for each
// of its first `bins` bins, the bin's segments in order, each cut into its
// full tiles and at most one remainder, then the end offsets of the bin.
// row_arena_offset[row] is the arena element offset of the key on that
// row.  Returns the number of elements scheduled, or -1 (nothing usable
// appended) when a table outgrows 32-bit offsets.
int64_t append_device_tables(const Plan& plan, const std::vector<VirtualKey>& vkeys,
                             const std::vector<int64_t>& row_arena_offset, int bins,
                             DeviceTables* out);

// How the tiles of the launch whose block of 2 * bins + 1 offsets starts at
// `block` in dt.tile_begin lie on its waves.
TileLoad tile_load(const DeviceTables& dt, size_t block, int bins, int64_t waves);

// Sets the calling thread's error message (phub_last_error) and returns code.
int report_error(int code, const std::string& message);

// Appends the WaveHead of each of `bins` waves of one launch whose block of
// 2 * bins + 1 bin offsets starts at `block` in dt.tile_begin and
// dt.rem_begin (the resident bins, then the streamed ones).
void append_wave_heads(const DeviceTables& dt, size_t block, int bins,
                       std::vector<WaveHead>* out);

// Enqueues one fused aggregate + optimize pass over the whole schedule
// (and, when p.outs is set, writes the updated weights into every worker's
// model buffer in the same pass; when p.merge is set, runs the unfused
// two-pass ablation instead): `grid` workgroups of kBlockThreads threads,
// two bins per wave as described above.  `optimizer` is an OptKind.
hipError_t launch_fused_step(const StepParams& p, int optimizer, int grid, hipStream_t stream);

// Loads per block where a step's streamed tiles are walked as one stream of
// load blocks (stream_walk.hpp), 5 or 6; 0: the fixed-N kernels' window over
// a tile is faster.  Measured on MI355X with nothing cached, 25.6 and 61.1 M
// parameters, fraction of peak, window over a tile -> stream (the better of
// the two blocks):
//   momentum  8 workers 0.827 -> 0.842, 9 0.827 -> 0.849, 13 0.834 -> 0.838,
//             14 0.837 -> 0.852, 15 0.837 -> 0.856, 16 0.838 -> 0.850,
//             20 0.845 -> 0.865, 24 0.847 -> 0.854, 32 0.837 -> 0.868, 10
//             +0.2 to +0.7 points; 7, 11 and 12 0.4 to 1.4 points below
//   SGD       9 0.839 -> 0.853, 10 0.845 -> 0.867, 11 0.851 -> 0.857, 15
//             0.851 -> 0.865, 16 0.852 -> 0.872, 24 0.860 -> 0.870, 32 0.859
//             -> 0.867; 7, 8 and 12 0.3 to 1 point below, 13 and 14 level
//   Adam      7 0.768 -> 0.790, 8 0.757 -> 0.806, 10 0.720 -> 0.791, 12 0.747
//             -> 0.811, 14 0.784 -> 0.825, 16 0.773 -> 0.819, 32 0.798 ->
//             0.846
// With 6 workers and fewer a piece would be a single block.
constexpr int kStreamBlock[3][kMaxFixedWorkers] = {
    {0, 0, 0, 0, 0, 0, 0, 0, 5, 5, 6, 0, 0, 0, 6, 6},
    {0, 0, 0, 0, 0, 0, 0, 5, 5, 6, 0, 0, 6, 5, 6, 6},
    {0, 0, 0, 0, 0, 0, 5, 5, 6, 5, 5, 5, 6, 5, 6, 6},
};

// Fewest streamed tiles per wave for that: the stream starts slower (a
// descriptor, then pointers, then data, where the other kernels' first
// descriptors come with the head).  Stream against window over a tile at 2,
// 3, 4, 5, 6 and 8 tiles per wave: momentum with 8 workers -1.8, -1.6, 0.0,
// -0.1, +1.1, +0.3 points, 16 workers +0.6, +0.3, -0.7, +1.0, +0.3, +1.4;
// SGD with 10 -0.3, +0.9, +0.4, +1.3, +2.2, +2.3; Adam with 8 +1.5, +1.9,
// +2.9, +4.9, +3.9, +3.9; below one tile 4 to 12 points down (momentum).
constexpr int kStreamMinTiles[3] = {4, 4, 2};

constexpr int stream_block(int num_workers, int num_states) {
    return num_workers > kMaxFixedWorkers ? 6 : kStreamBlock[num_states - 1][num_workers - 1];
}

// When a dealt schedule (build_dealt) cuts the tiles left over from the last
// whole round evenly over the waves.  Measured on MI355X, whole -> cut.
// From one round on, where the state is streamed and written back in bursts:
// 8 workers over 1.2 M parameters 12.2 -> 10.8 us, over 4.7 M 39.3 -> 37.4, 16
// over 2.4 M 34.7 -> 32.4, pushpull with 8 over 1.2 M 23.0 -> 20.7, Adam with
// 7 over 2.4 M 25.9 -> 24.3.  Without bursts a wave runs a second tile on in
// the load window of the first, and a piece costs its own trip to memory: 2
// workers over 1.2 M 6.8 -> 7.6 us, 4 over 1.2 M 8.3 -> 9.1, Adam with 8 over
// 1.7 M 19.4 -> 20.4, cached state with 8 over 1.2 M 11.4 -> 12.5; four jobs at
// once up to 25% (1 worker, Adam, 1.7 M each 37 -> 46).  From 16 rounds on it
// is level to 2% faster, pushpull 1 to 3%, four jobs at once within 1%; with as
// many workers as bursts take, cached state reaches that at 4 rounds (pushpull
// with 8 over 5.6 M 77.0 -> 74.0).  The any-N stream's piece is a walk of its
// own (17 workers over 1.4 M 23.2 -> 24.4): below eight rounds 0 to 5% slower,
// beyond within 1% either way, alone up to 1% faster (64 workers over 25.6 M
// 1024 -> 1016).
// Below one round most waves would have no tile.  Pieces of up to half a tile
// gain up to 1.6 times (Adam with 8 over 0.4 M 8.4 -> 6.5 us, 16 workers over
// 0.4 M 9.2 -> 6.3, 64 over 0.02 M 15.0 -> 9.7) and cost four jobs at once 0
// to 6%, at worst 19; longer ones gain 0 to 7% (cached state up to 15) with as
// many workers as bursts take, else less than they cost jobs that run at the
// same time (two of 8 workers over 0.6 M each 9.3 -> 10.2 us).
constexpr Cut cut_rule(int num_workers, int num_states, bool streamed, bool unfused) {
    const bool fixed = has_fixed_kernel(num_workers) && !unfused;
    const bool burst = fixed && burst_write_back(num_workers, num_states);
    Cut cut;
    cut.below_one_round = burst ? kTileElems * 3 / 4 : kTileElems / 2;
    cut.rounds = 16;
    if (burst)
        cut.rounds = streamed ? 0 : 4;
    else if (streamed && fixed && stream_block(num_workers, num_states) != 0)
        cut.rounds = kStreamMinTiles[num_states - 1];
    else if (streamed && !unfused && !fixed)
        cut.rounds = 8;
    return cut;
}

// Whether a step of a fixed-N kernel walks its streamed tiles as one stream
// (no model buffers; grid_waves: the launch's waves).  Not where chunks kept
// whole leave waves idle: over 5 M parameters in 32 KB chunks (five waves of
// eight busy at the end) the stream was level to 4% below the window over a
// tile for momentum and plain SGD (SGD with 9 workers 48.2 -> 50.5 us), over
// 25 M up to 3% above; for Adam it was level to 12% above on both.
constexpr bool takes_stream(int num_workers, int num_states, const TileLoad& l,
                            int64_t grid_waves) {
    return has_fixed_kernel(num_workers) && stream_block(num_workers, num_states) != 0 &&
           l.streamed >= kStreamMinTiles[num_states - 1] * grid_waves &&
           (num_states == 3 || 4 * (l.streamed + l.resident) >= 3 * l.busiest * grid_waves);
}

// The kernel of a step (no model buffers) without a fixed-N kernel: batches
// of workers' loads issued and drained (fused_step_any), or the stream walk
// (fused_step_many), whose pieces take at least two blocks of loads.
enum AnyKernel { kAnyBatches, kAnyStream, kAnyStreamShared };
constexpr int kManyBlock = 6;  // loads of a block

// The stream walk keeps six loads in flight per wave, a batch thirty-two: the
// stream is the faster where the launch's waves share the work, the batches
// where a few of them have most of it (chunks kept whole) and each waits for
// memory's latency.  The share of the waves that is busy until the busiest
// ends, batches -> stream (17 to 64 workers, the three optimizers): 1/8
// 0.78-0.85 of the speed, 1/4 0.81-0.88, 1/2 0.94-1.0, 5/8 0.92-0.99, 3/4
// 1.01-1.07, 7/8 1.09-1.14.  Up to two tiles a wave the schedules that
// phub_init deals are never uneven in that sense; and many small keys are the
// stream's (31 workers over 0.5 M parameters in 443 keys, chunks kept whole,
// 190 -> 145 us).  A grid of few workgroups is not counted: it is for tenants
// to share the chip, where the stream is the faster (four of 21 workers over
// 25.6 M on 64 workgroups each 2511 -> 2244 us, though one alone on 64, 94
// workers over 1.9 M, 272 -> 300).
constexpr bool few_waves_busy(const TileLoad& l) {
    const int64_t tiles = l.streamed + l.resident;
    return l.busiest > 2 && tiles >= l.rems && 8 * tiles <= 5 * l.busiest * l.waves;
}

// State that is cached needs no bursts.  Up to three tiles a wave the stream
// is still the faster, by what a launch's ends weigh there; its stash, small
// enough that tenants share a compute unit (fused_many_shared.hip), is for
// the loads not to wait for stores.  With more tiles the batches are level or
// faster.  Batches -> stream, the speed of one job and of four at once (17 to
// 64 workers, the three optimizers): 1 tile 1.32-1.44 and 0.99-1.15, 2 tiles
// 1.11-1.22 and 0.95-1.02, 3 tiles 0.99-1.16 and 0.98-1.07, 4 tiles
// 0.96-1.09 and 0.98-1.05, 25.6 M parameters with 21 0.97 (one job).  (Tiles
// per wave of the device: a larger grid splits the same work.)
constexpr int64_t kSharedTiles = 3;
constexpr int kSharedStashBytesPerWave = 16 * 1024;
constexpr int shared_stash_tiles(int num_states) {
    return kSharedStashBytesPerWave / (num_states * 4 * 1024);
}

constexpr AnyKernel any_kernel(int num_workers, const TileLoad& load) {
    if (num_workers <= kManyBlock || few_waves_busy(load)) return kAnyBatches;
    if (load.resident >= load.streamed)  // (none of either: remainders only)
        return load.resident + load.streamed <= kSharedTiles * load.waves ? kAnyStreamShared
                                                                          : kAnyBatches;
    return kAnyStream;
}

// The fused pass of launch_fused_step with fused_step_many, its whole stash or
// the shared one: more than kManyBlock workers (no model buffers, no merge
// buffer, no pool).
hipError_t launch_fused_step_many(const StepParams& p, int optimizer, int grid,
                                  hipStream_t stream);
hipError_t launch_fused_step_many_shared(const StepParams& p, int optimizer, int grid,
                                         hipStream_t stream);

// The same for worker counts with a fixed-N kernel where stream_block is not
// 0 (OPT an OptKind).
template <int OPT>
hipError_t launch_stream(const StepParams& p, int grid, hipStream_t stream);

// Enqueues the writing of up to kPutPointers pointers to the device address
// dst as the arguments of one launch (`pointers` may change once it
// returns); false, with nothing enqueued, where there are more or one does
// not fit 48 bits.
constexpr int kPutPointers = 640;
bool put_pointers(const void* const* pointers, size_t count, void* dst, hipStream_t stream,
                  hipError_t* error);

}  // namespace phub
