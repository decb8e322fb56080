// Host-only check of the rules by which libdear chooses launches (dear_internal.h).  Exits non-zero on the first
// broken one.
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "dear_internal.h"

#define CHECK(c)                                                         \
    do {                                                                 \
        if (!(c)) {                                                      \
            std::fprintf(stderr, "FAILED %s (line %d)\n", #c, __LINE__); \
            std::exit(1);                                                \
        }                                                                \
    } while (0)

static bool hip_takes(int64_t workgroups) { return workgroups >= 1 && workgroups * DEAR_BLOCK < (int64_t(1) << 32); }

static void grids()
{
    CHECK(hip_takes(MAX_GRID) && !hip_takes(MAX_GRID + 1));
    static const int64_t workers[] = {1, 2, 5, 6, 7, 8, 64, 1000, 4096, 23170, 70000};
    static const int64_t widths[] = {0, 1, 256, 100000, MAX_GRID, MAX_GRID + 1, 0x7fffffff};
    for (int64_t P : workers)
        for (int64_t width : widths) {
            const int64_t at[] = {1, UAG_SPLIT_TILES / P, MAX_GRID / (AG_SPLIT * P), 0x3fffffff / (AG_SPLIT * P),
                                  0x7fffffff / (AG_SPLIT * P), 300000, 0x7fffffff / 16};
            for (int64_t middle : at)
                for (int64_t tiles = middle > 2 ? middle - 2 : 1; tiles <= middle + 2; ++tiles) {
                    const int64_t items = tiles * AG_SPLIT * P;
                    const bool bounded = all_gather_bounded(tiles, P, width);
                    const bool fits = all_gather_fits(tiles, P, width);
                    // the grid that launch_all_gather asks for
                    if (fits) CHECK(hip_takes(!bounded ? items : width < tiles ? width : tiles));
                    if (!bounded) CHECK(fits == hip_takes(items));
                    if (bounded && width <= MAX_GRID) CHECK(fits == (items <= 0x7fffffff));
                    // the update goes first, so the all-gather behind it must be one that can be launched
                    if (update_all_gather_splits(tiles, P, width)) {
                        CHECK(fits && P >= UAG_SPLIT_P && tiles * P >= UAG_SPLIT_TILES);
                        CHECK(width <= 0 || tiles <= width);
                    }
                }
        }
    // 268 M elements in one call for 64 workers: the all-gather's grid is 2^24 workgroups, the one kernel's 65536
    CHECK(update_all_gather_splits(65535, 64, 0) && !update_all_gather_splits(65536, 64, 0));
    CHECK(!all_gather_fits(65536, 64, 0) && all_gather_fits(65536, 64, 256));
}

int main()
{
    grids();
    std::printf("launch_rules: ok\n");
    return 0;
}
