// The choice of the any-N kernel and of the stream walk of the fixed-N kernels
// on the host.  Exit status 0 when all hold.
#include <cstdio>
#include <cstdlib>
#include <utility>
#include <vector>

#include "kernels.hpp"

using namespace phub;

static void check(bool ok, const char* what, int64_t a = 0, int64_t b = 0) {
    if (ok) return;
    std::fprintf(stderr, "%s (%lld, %lld)\n", what, (long long)a, (long long)b);
    std::exit(1);
}

// The load of `keys` dealt over `bins` of a device of `waves` waves.
static TileLoad dealt(const std::vector<int64_t>& keys, int bins, int64_t waves) {
    Plan p;
    if (!build_dealt(int(keys.size()), keys.data(), kTileElems, 100, bins, &p, Cut{1 << 30, 0}).empty()) std::exit(2);
    TileLoad l{0, 0, 0, 0, waves};
    for (int b = 0; b < bins; ++b) {
        int64_t tiles = 0;
        for (int64_t i = p.bin_begin[b]; i < p.bin_begin[b + 1]; ++i) {
            tiles += p.segments[i].count / kTileElems;
            l.rems += p.segments[i].count % kTileElems != 0;
        }
        l.streamed += tiles;
        l.busiest = tiles > l.busiest ? tiles : l.busiest;
    }
    return l;
}

int main() {
    const int64_t waves = 1024;
    // a piece of the stream walk takes at least two blocks: never below
    for (int n = 1; n <= kMaxWorkers; ++n)
        check((any_kernel(n, {50 * waves, 0, 0, 50, waves}) == kAnyBatches) == (n <= kManyBlock), "workers", n);
    // jobs of the default schedule on the default grid share the chip's waves
    for (int64_t elems : {1, 1000, 500000, 1048576, 1050000, 1300000, 2097152, 2100000, 3145728,
                          3200000, 5000000, 25557032}) {
        TileLoad l = dealt({elems, 77, 301}, int(waves), waves);
        check(any_kernel(17, l) == (l.streamed ? kAnyStream : kAnyStreamShared), "dealt", elems);
        // the same with its state cached, whole and by halves
        std::swap(l.streamed, l.resident);
        check(any_kernel(17, l) == (l.resident <= 3 * waves ? kAnyStreamShared : kAnyBatches), "cached",
              elems);
        l.streamed = l.resident;
        check(any_kernel(17, l) == (2 * l.resident <= 3 * waves ? kAnyStreamShared : kAnyBatches), "half",
              elems);
        l.streamed = l.resident + 1;
        check(any_kernel(17, l) == kAnyStream, "mostly streamed", elems);
    }
    for (int s : {1, 2, 3})  // two launches' workgroups fit a compute unit
        check(shared_stash_tiles(s) >= 1 &&
                  2 * 4 * shared_stash_tiles(s) * s * 4096 <= 160 * 1024, "shared stash", s);
    // chunks of 8 tiles kept whole: items each on a wave of its own, or two
    for (int64_t items : {1, 3, 128, 512, 640})
        check(any_kernel(33, {8 * items, 0, 0, 8, waves}) == kAnyBatches, "few whole chunks", items);
    for (int64_t items : {768, 1024, 1536, 5000})
        check(any_kernel(33, {8 * items, 0, 0, 8 * ((items + waves - 1) / waves), waves}) == kAnyStream,
              "whole chunks", items);
    // the same with more small keys than tiles
    check(any_kernel(33, {8 * 128, 0, 8 * 128 + 1, 8, waves}) == kAnyStream, "small keys");
    // a grid of any size
    for (int grid : {1, 32, 64, 128, 160, 192, 224, 256, 512})
        check(any_kernel(64, dealt({4000000}, 4 * grid, 4 * (grid < 256 ? grid : 256))) == kAnyStream,
              "grid", grid);
    // the fixed-N kernels' stream walk: enough streamed tiles for the launch's
    // waves, and for momentum and plain SGD evenly spread
    for (int s : {1, 2, 3})
        for (int n = 1; n <= 40; ++n) {
            const bool stream = has_fixed_kernel(n) && stream_block(n, s) != 0;
            const int64_t least = kStreamMinTiles[s - 1];
            for (int64_t g : {4, 12, 1024}) {
                check(takes_stream(n, s, {least * g, 0, 0, least, waves}, g) == stream, "least", n, s);
                check(!takes_stream(n, s, {least * g - 1, 0, 0, least, waves}, g), "fewer", n, s);
                check(takes_stream(n, s, {20 * g, 0, 0, 26, waves}, g) == stream, "even", n, s);
                check(takes_stream(n, s, {20 * g, 0, 0, 27, waves}, g) == (stream && s == 3), "uneven", n, s);
                check(!takes_stream(n, s, {0, 90 * g, 0, 90, waves}, g), "cached", n, s);
            }
            // the grids on which tests/test_gpu_stream_kernels.py means the stream
            // walk, and those on which it means the window over a tile
            const std::vector<int64_t> keys = {5, 1024 * 37 + 3, 70001, 1024 * 11, 4097, 1, 1024 * 6};
            check(takes_stream(n, s, dealt(keys, 4, waves), 4) == stream, "one workgroup", n, s);
            const int few = s == 3 ? 64 : 40;
            check(!takes_stream(n, s, dealt(keys, few, waves), few), "few tiles", n, s);
            // what phub_init deals is even, cut or not
            for (int64_t elems : {4200000, 5000000, 6400000, 25557032})
                check(takes_stream(n, s, dealt({elems, 77, 301}, int(waves), waves), waves) == stream,
                      "dealt", n, elems);
        }
    return 0;
}
