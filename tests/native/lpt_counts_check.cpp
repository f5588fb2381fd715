// lpt_counts (the tiles and remainders of a schedule counted key by key)
// against build_plan's own segments, over edge and random key lists, chunk
// sizes and item minimums.  Exit status 0 when all agree.
#include <cstdio>
#include <random>
#include <vector>

#include "plan.hpp"

int main() {
    std::mt19937_64 rng(1805);
    std::vector<std::vector<int64_t>> lists = {
        {0}, {1}, {0, 0, 5}, {1023, 1024, 1025}, {100, 0, 100, 9000, 100, 100}, {8192, 8191, 8193, 1}};
    for (int i = 0; i < 300; ++i) {
        std::vector<int64_t> keys(1 + rng() % 60);
        for (auto& n : keys) n = int64_t(rng() % (uint64_t(1) << (rng() % 19))) * (rng() % 8 != 0);
        lists.push_back(keys);
    }
    const int64_t tile = 1024;
    long checked = 0;
    for (const auto& keys : lists)
        for (int64_t chunk : {16, 4000, 4096, 4112, 32768, 1 << 20})
            for (int min_items : {0, 3, 100, 131072}) {
                phub::Plan plan;
                const std::string err =
                    phub::build_plan(4, int(keys.size()), keys.data(), chunk, phub::kScheduleLpt, 64,
                                     min_items, &plan);
                if (!err.empty()) return 2;
                int64_t tiles = 0, rems = 0;
                for (const auto& s : plan.segments) {
                    tiles += s.count / tile;
                    rems += s.count % tile != 0;
                }
                const phub::LptCounts c =
                    phub::lpt_counts(int(keys.size()), keys.data(), chunk, min_items, tile);
                if (c.tiles != tiles || c.rems != rems) {
                    std::fprintf(stderr, "%zu keys, chunk %lld, min_items %d: %lld %lld, want %lld %lld\n",
                                 keys.size(), (long long)chunk, min_items, (long long)c.tiles,
                                 (long long)c.rems, (long long)tiles, (long long)rems);
                    return 1;
                }
                ++checked;
            }
    std::printf("%ld schedules\n", checked);
    return 0;
}
