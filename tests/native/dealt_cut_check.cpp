// Where build_dealt and the rule of phub_init cut the tiles left over from
// the last round: only from the rounds asked for, and then spread evenly; the rule asks for streamed state written back in bursts,
// from eight rounds on without a fixed-N kernel.  Exit status 0 when all
// hold.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "kernels.hpp"

static void check(bool ok, const char* what, int64_t tiles, int bins) {
    if (ok) return;
    std::fprintf(stderr, "%lld tiles, %d bins: %s\n", (long long)tiles, bins, what);
    std::exit(1);
}

int main() {
    const int64_t tile = phub::kTileElems;
    int cut_plans = 0;
    for (int bins : {1, 8, 1024})
        for (int64_t tiles : {1, 4, 7, 8, 9, 586, 1023, 1024, 1025, 1327, 1500, 2047, 2048, 4600, 9000})
            for (int rounds : {-1, 0, 1, 8}) {
                const std::vector<int64_t> keys = {tiles / 2 * tile, (tiles - tiles / 2) * tile + 5};
                phub::Plan p;
                if (!phub::build_dealt(2, keys.data(), tile, 48, bins, &p, rounds).empty()) return 2;
                int64_t pieces = 0;
                for (const auto& s : p.segments)
                    pieces += s.count != tile && s.count != 5;
                const bool may = rounds >= 0 && tiles / bins >= rounds && tiles % bins != 0;
                check(may || pieces == 0, "cut", tiles, bins);
                check(pieces > 0 || int64_t(p.segments.size()) == tiles + 1, "segments", tiles, bins);
                if (pieces) {
                    ++cut_plans;
                    for (int b = 0; b < bins; ++b)
                        // (each of the two keys may leave a short last piece)
                        check(p.bin_begin[b + 1] - p.bin_begin[b] <= tiles / bins + 2, "spread",
                              tiles, bins);
                }
            }
    check(cut_plans > 0, "no plan was cut", 0, 0);
    for (int n = 1; n <= 70; ++n)
        for (int s : {1, 2, 3}) {
            const int want = !phub::has_fixed_kernel(n) ? 8 : phub::burst_write_back(n, s) ? 0 : -1;
            check(phub::cut_rounds(n, s, true, false) == want, "rule: streamed", n, s);
            check(phub::cut_rounds(n, s, false, false) < 0, "rule: cached", n, s);
            check(phub::cut_rounds(n, s, true, true) < 0, "rule: unfused", n, s);
        }
    std::printf("%d cut\n", cut_plans);
    return 0;
}
