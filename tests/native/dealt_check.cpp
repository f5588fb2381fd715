// build_dealt over edge and random key lists and bin counts: every element
// covered exactly once by segments that start on a 16-byte boundary, no
// segment above a tile, bins in key and offset order, costs added up, and
// the list-scheduling bound (average load plus the largest item); what is
// cut is cut only where it gives every bin less than a tile more.  Exit
// status 0 when all hold.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <vector>

#include "plan.hpp"

static void check(bool ok, const char* what, size_t list, int bins) {
    if (ok) return;
    std::fprintf(stderr, "list %zu, %d bins: %s\n", list, bins, what);
    std::exit(1);
}

int main() {
    const int64_t tile = 1024, per = 48;
    std::mt19937_64 rng(1805);
    std::vector<std::vector<int64_t>> lists = {{0}, {1}, {0, 5, 0}, {1023, 1024, 1025, 0},
                                               {1024 * 7}, {1024 * 1024 * 3 + 4}, {1 << 20, 1 << 20}};
    for (int i = 0; i < 150; ++i) {
        std::vector<int64_t> keys(1 + rng() % 400);
        for (auto& n : keys) n = int64_t(rng() % (uint64_t(1) << (rng() % 20))) * (rng() % 9 != 0);
        lists.push_back(keys);
    }
    long plans = 0;
    for (size_t li = 0; li < lists.size(); ++li)
        for (int bins : {1, 4, 12, 1024, 3000}) {
            const auto& keys = lists[li];
            phub::Plan p;
            check(phub::build_dealt(int(keys.size()), keys.data(), tile, per, bins, &p).empty(),
                  "error", li, bins);
            check(int(p.bin_begin.size()) == bins + 1 && p.bin_begin[0] == 0 &&
                      p.bin_begin[bins] == int64_t(p.segments.size()), "bin offsets", li, bins);
            std::vector<std::map<int64_t, int64_t>> seen(keys.size());
            int64_t total = 0, largest = 0, worst = 0;
            for (int b = 0; b < bins; ++b) {
                int64_t cost = 0;
                for (int64_t i = p.bin_begin[b]; i < p.bin_begin[b + 1]; ++i) {
                    const auto& s = p.segments[i];
                    check(s.count >= 1 && s.count <= tile && s.offset % 4 == 0, "segment", li, bins);
                    check(seen[s.key].emplace(s.offset, s.count).second, "twice", li, bins);
                    if (i > p.bin_begin[b]) {
                        const auto& q = p.segments[i - 1];
                        check(q.key < s.key || (q.key == s.key && q.offset < s.offset), "order", li, bins);
                    }
                    const int64_t c = s.count * per + phub::kSegmentCostBytes;
                    cost += c;
                    largest = std::max(largest, c);
                }
                check(cost == p.bin_cost[b], "cost", li, bins);
                total += cost;
                worst = std::max(worst, cost);
            }
            check(worst <= total / bins + 1 + largest, "balance", li, bins);
            for (size_t k = 0; k < keys.size(); ++k) {
                int64_t at = 0;
                for (const auto& [off, count] : seen[k]) {
                    check(off == at, "gap or overlap", li, bins);
                    at = off + count;
                }
                check(at == keys[k], "coverage", li, bins);
            }
            ++plans;
        }
    std::printf("%ld plans\n", plans);
    return 0;
}
