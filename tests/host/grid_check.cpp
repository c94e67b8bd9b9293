// Host-side checks of the launch rules whose index space can pass the 2^32
// work-items of a dispatch: every size the library accepts stays below it.
#include "internal.h"

#include <cstdio>
#include <cstdlib>

using namespace rrt;

static void below(const char* what, int64_t a, double b, double items)
{
    if (items >= 1.0 && items < 4294967296.0) return;
    std::fprintf(stderr, "%s(%lld, %g): %.0f work-items\n", what, (long long)a, b, items);
    std::exit(1);
}

int main()
{
    for (int e = 0; e <= 27; ++e)
        for (int d = -1; d <= 1; ++d) {
            const int64_t n = (int64_t(1) << e) + d;
            if (n < 1 || n > (int64_t(1) << 27)) continue;
            for (int bins : {1, 63, 64, 65, 256, 2048, kMaxBins})
                below("adj_wbins_blocks", n, bins, 256.0 * adj_wbins_blocks(n, bins));
        }
    // packets: at most kMaxRows rays, and one more short packet per direction
    for (int64_t pk : {int64_t(1), int64_t(16383), int64_t(16384), int64_t(663552),
                       int64_t(1) << 22, int64_t(1) << 23, int64_t(1) << 24, int64_t(1) << 25,
                       kMaxRows / 64 + kMaxRays})
        for (uint64_t segs : {0, 1, 4, 7, 13, 25, 1000000})
            for (int64_t live : {int64_t(0), int64_t(1), pk / 3, pk})
                below("path_ways", pk, (double)segs,
                      (double)pk * 64.0 * path_ways(pk, live, segs * (uint64_t)live));
    // the measured choices
    if (path_ways(663552, 663552, 2256077) != 2 || path_ways(49152, 49152, 983040) != 4 ||
        path_ways(26236, 26236, 236124) != 2 || path_ways(100, 100, 900) != 8 ||
        path_ways(100, 100, 100) != 1 || path_ways(936, 250, 900) != 4) {
        std::fprintf(stderr, "path_ways: not the measured choices\n");
        return 1;
    }
    // packets that are not recorded: their waves count against the gain
    if (path_ways(1335724, 667862, 13357240) != 2 || path_ways(1335724, 250, 5000) != 1 ||
        path_ways(26236, 8745, 78705) != 2) {
        std::fprintf(stderr, "path_ways: packets that are not recorded do not count\n");
        return 1;
    }
    std::printf("grid checks passed\n");
    return 0;
}
