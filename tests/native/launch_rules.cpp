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
                    int64_t grid = width < tiles ? width : tiles;
                    if (!bounded && fits) {
                        const unsigned parts = static_cast<unsigned>(tiles * AG_SPLIT), whole = parts / 4096 * 4096;
                        grid = (int64_t(whole) + all_gather_numbering(2, width, whole, parts, P).len) * P;
                        CHECK(grid >= items && (width <= 0 || grid <= width));
                    }
                    if (fits) CHECK(hip_takes(grid));
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

// Bounding the workgroups per CU pays only in long launches of full tiles.
static void residency()
{
    for (int bf16 = 0; bf16 < 2; ++bf16)
        for (int updates = 0; updates < 2; ++updates)
            for (int64_t P = 1; P <= 70; ++P) {
                int before = 0;
                for (int64_t elems = 1000; elems < int64_t(1) << 37; elems *= 2) {
                    const int64_t full = elems / DEAR_TILE_ELEMS + 1;
                    const int r = reduce_scatter_residency(bf16, updates, P, elems, full);
                    CHECK(r == 0 || ((r == 2 || (r == 1 && bf16)) && elems * P * (bf16 ? 2 : 4) >= 160000000));
                    if (P < 4) CHECK(r == 0);
                    CHECK(before == 0 || (r != 0 && r <= before));  // longer launches: the same bound or a tighter one
                    before = r;
                    // the same elements in runs of 3000: three quarters full
                    CHECK(reduce_scatter_residency(bf16, updates, P, elems, elems / 3000 + 1) == 0);
                }
            }
    struct { bool bf16, updates; int64_t P, elems; int want; } const at[] = {
        {false, true, 4, 31200000, 0},   {false, true, 4, 31300000, 2},   {false, true, 3, 110000000, 0},
        {false, true, 8, 12400000, 0},   {false, true, 8, 12600000, 2},
        {false, false, 4, 110000000, 0}, {false, false, 8, 24900000, 0},  {false, false, 8, 25100000, 2},
        {false, false, 16, 6200000, 0},  {false, false, 16, 6300000, 2},  {true, true, 5, 15900000, 0},
        {true, true, 5, 110000000, 2},   {true, true, 8, 28700000, 2},    {true, true, 8, 28800000, 1},
        {true, false, 8, 110000000, 2},  {true, false, 16, 15600000, 0},  {true, false, 16, 15700000, 1},
        {true, false, 12, 110000000, 2}, {true, false, 20, 110000000, 2}, {true, false, 17, 110000000, 1},
    };
    for (const auto &c : at)
        CHECK(reduce_scatter_residency(c.bf16, c.updates, c.P, c.elems, c.elems / DEAR_TILE_ELEMS + c.P) == c.want);
}

// dear_iteration: w is left in the cache only where it fits; gbar is read again only where many replicas are read.
static void iteration()
{
    for (int g = 2; g <= 4; g += 2)
        for (int64_t P = 1; P <= 80; ++P)
            for (int64_t tiles : {int64_t(1), int64_t(2047), int64_t(2048), ITERATION_TILES, ITERATION_TILES + 1, int64_t(100000)})
                for (int64_t all : {tiles, tiles + 1, 2 * tiles + 7168}) {
                    const bool cached = iteration_caches_w(g, P, tiles, all), apart = iteration_updates_apart(g, P, tiles);
                    CHECK(!cached || tiles <= ITERATION_TILES);
                    CHECK(!cached || g * P <= (g == 2 ? 24 : 16) || (g * P <= 64 && all <= 7168));
                    CHECK(cached || tiles > ITERATION_TILES || g * P > (g == 2 ? 24 : 16));
                    CHECK(apart == (g * P >= 96 && tiles >= 2048));
                    CHECK(!(apart && cached));
                }
}

int main()
{
    grids();
    residency();
    iteration();
    std::printf("launch_rules: ok\n");
    return 0;
}
