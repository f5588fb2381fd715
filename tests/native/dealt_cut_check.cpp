// Where build_dealt and the rule of phub_init cut the tiles left over from
// the last round: only from the rounds asked for, below one round only into
// pieces as short as asked for, and spread evenly; the rule against its
// classes of jobs.  Exit status 0 when all hold.
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
    using phub::Cut;
    const int64_t tile = phub::kTileElems;
    int cut_plans = 0;
    for (int bins : {1, 8, 1024})
        for (int64_t tiles : {1, 3, 4, 7, 8, 9, 400, 586, 1023, 1024, 1025, 1327, 1500, 2047, 2048, 4600, 9000})
            for (const Cut cut : {Cut{1 << 30, 0}, Cut{16, 512}, Cut{0, 768}, Cut{1, 512}, Cut{8, 512}}) {
                const std::vector<int64_t> keys = {tiles / 2 * tile, (tiles - tiles / 2) * tile + 5};
                phub::Plan p;
                if (!phub::build_dealt(2, keys.data(), tile, 48, bins, &p, cut).empty()) return 2;
                int64_t pieces = 0, longest = 0;
                for (const auto& s : p.segments)
                    if (s.count != tile && s.count != 5) {
                        ++pieces;
                        longest = s.count > longest ? s.count : longest;
                    }
                const bool below = tiles < bins;
                const bool may = below ? cut.below_one_round > 0
                                       : tiles / bins >= cut.rounds && tiles % bins != 0;
                check(may || pieces == 0, "cut", tiles, bins);
                check(longest <= (below ? cut.below_one_round : 768), "piece", tiles, bins);
                check(pieces > 0 || int64_t(p.segments.size()) == tiles + 1, "segments", tiles, bins);
                if (pieces) {
                    ++cut_plans;
                    for (int b = 0; b < bins; ++b)
                        // (each of the two keys may leave a short last piece)
                        check(p.bin_begin[b + 1] - p.bin_begin[b] <= tiles / bins + 2, "spread",
                              tiles, bins);
                }
                // a piece of half a tile or less is always worth it below one round
                if (bins == 1024 && tiles == 400) check((pieces > 0) == may, "short pieces", tiles, bins);
            }
    check(cut_plans > 0, "no plan was cut", 0, 0);
    for (int n = 1; n <= 70; ++n)
        for (int s : {1, 2, 3}) {
            const bool fixed = phub::has_fixed_kernel(n), burst = fixed && phub::burst_write_back(n, s);
            const bool adam_stream = fixed && s == 3 && n >= 7 && !burst;
            const Cut c = phub::cut_rule(n, s, true, false);
            check(c.rounds == (!fixed ? 8 : burst ? 0 : adam_stream ? 2 : 16), "rule: streamed", n, s);
            check(c.below_one_round == (burst ? 768 : 512), "rule: short", n, s);
            check(phub::cut_rule(n, s, false, false).rounds == (burst ? 4 : 16), "rule: cached", n, s);
            check(phub::cut_rule(n, s, false, false).below_one_round == c.below_one_round, "rule: cached", n, s);
            check(phub::cut_rule(n, s, true, true).rounds == 16, "rule: unfused", n, s);
        }
    std::printf("%d cut\n", cut_plans);
    return 0;
}
