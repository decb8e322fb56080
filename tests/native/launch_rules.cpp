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
            const int64_t at[] = {1, 4096 / P, MAX_GRID / (AG_SPLIT * P), 0x3fffffff / (AG_SPLIT * P),
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
                        grid = (int64_t(whole) + all_gather_numbering(1, width, whole, parts, P).len) * P;
                        CHECK(grid >= items && (width <= 0 || grid <= width));
                    }
                    if (fits) CHECK(hip_takes(grid));
                    if (!bounded) CHECK(fits == hip_takes(items));
                    if (bounded && width <= MAX_GRID) CHECK(fits == (items <= 0x7fffffff));
                    // the update goes first, so the all-gather behind it must be one that can be launched
                    for (int64_t elems : {tiles * DEAR_TILE_ELEMS, tiles * 3500})
                        if (update_all_gather_splits(elems, tiles, elems / DEAR_TILE_ELEMS, P, width)) {
                            CHECK(fits && P >= UAG_SPLIT_P && elems * P >= 15600000 && elems >= 920000);
                            CHECK(width <= 0 || tiles <= width);
                        }
                }
        }
    // 268 M elements in one call for 64 workers: the all-gather's grid is 2^24 workgroups, the one kernel's 65536
    CHECK(update_all_gather_splits(65535ll << 12, 65535, 65535, 64, 0) && !update_all_gather_splits(65536ll << 12, 65536, 65536, 64, 0));
    CHECK(!all_gather_fits(65536, 64, 0) && all_gather_fits(65536, 64, 256));
}

// bf16 reduce-scatters in half tiles: short launches, some of whose tiles are whole or which are a quarter (many: three eighths) full.
static void half_tiles()
{
    CHECK(reduce_scatter_half_tiles(true, 0, 1024 * 4096, 1024, 1024) && !reduce_scatter_half_tiles(true, 0, 1025 * 4096, 1025, 1025));
    CHECK(reduce_scatter_half_tiles(false, 0, 160 * 4096, 160, 160) && !reduce_scatter_half_tiles(false, 0, 161 * 4096, 161, 161));
    for (bool updates : {false, true}) {
        CHECK(!reduce_scatter_half_tiles(updates, 256, 100 * 4096, 100, 100));
        CHECK(reduce_scatter_half_tiles(updates, 0, 100 * 1024, 100, 0) && !reduce_scatter_half_tiles(updates, 0, 100 * 1024 - 1, 100, 1));
        CHECK(reduce_scatter_half_tiles(updates, 0, 100 * 600, 100, 2));
    }
    CHECK(reduce_scatter_half_tiles(true, 0, 16, 16, 0) && !reduce_scatter_half_tiles(true, 0, 17, 17, 0));
    CHECK(reduce_scatter_half_tiles(true, 0, 200 * 1024, 200, 0) && !reduce_scatter_half_tiles(true, 0, 201 * 1536 - 1, 201, 0));
    CHECK(reduce_scatter_half_tiles(true, 0, 201 * 1536, 201, 0) && !reduce_scatter_half_tiles(true, 0, 406 * 1400, 406, 6));
    CHECK(reduce_scatter_half_tiles(true, 0, 406 * 1400, 406, 7));
}

// All-gathers in pairs of parts: where the bf16 reduce-scatter + update went in halves of tiles, and then mostly in dear_iteration.
static void pairs_of_parts()
{
    struct { int64_t P, tiles, fill; bool behind, apart; } const at[] = {
        {1, 40, 4000, true, true},   {8, 160, 2000, true, true},    {9, 160, 4000, true, false},   {9, 160, 3071, false, false}, {9, 160, 3072, true, false},
        {4, 161, 2000, true, true},  {5, 161, 4000, true, false},   {32, 399, 4000, true, false},  {33, 399, 4000, false, false}, {47, 400, 4000, true, false},
        {48, 400, 4000, false, false}, {4, 1024, 4000, true, true}, {8, 1024, 3000, true, false},  {8, 1025, 4000, true, false},
        {8, 2047, 4000, true, false},  {8, 2048, 4000, false, false}, {12, 1599, 4000, true, false}, {12, 1600, 4000, false, false},
        {13, 1025, 4000, false, false}, {13, 1024, 4000, true, false}, {4, 1025, 4000, true, false}, {4, 1025, 2048, true, false}, {4, 1025, 2047, false, false},
    };
    for (const auto &c : at) {
        const int64_t elems = c.tiles * c.fill;
        auto run = [&](int g, int64_t width, int64_t n, int64_t whole, bool behind) {
            return all_gather_run(g, behind, width, c.P, n, c.tiles, whole, c.tiles, 0, c.P, behind);
        };
        CHECK(run(2, 0, elems, c.tiles / 2, true) == c.behind);
        CHECK(run(2, 0, elems, c.tiles / 2, false) == c.apart);
        for (bool behind : {false, true}) {
            CHECK(run(4, 0, elems, c.tiles, behind) == 0);
            CHECK(run(2, 100000, elems, c.tiles, behind) == 0);
            CHECK(run(2, 0, c.tiles * 1000, 0, behind) == 0);
        }
    }
    // a reduce-scatter in whole tiles beyond 1024 of them: the batch kernel, in calls of its own
    CHECK(reduce_scatter_shape_of(true, true, false, 8, 1025 * 4096, 1025, 1025, 0).depth == 0);
    CHECK(all_gather_run(2, false, 0, 8, 1025 * 4096, 1025, 1025, 1025, 0, 8, true) == 0 && all_gather_run(2, true, 0, 8, 1025 * 4096, 1025, 1025, 1025, 0, 8, true) == 1);
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

// dear_update_all_gather: two launches from where they pay, by elements, replicas and open tiles.  (The limits of full tiles are
// those that test_gpu_parity.py's test of both sides takes.)  In one kernel: quarters of tiles in small launches, the smaller the more replicas, and in larger ones of
// few whole tiles among short ones.
static void update_and_gather()
{
    struct { int64_t P, tiles, fill, whole; bool quarters; } const at[] = {
        {1, 1, 5, 0, true},         {3, 112, 4096, 112, true},  {3, 113, 4096, 113, false}, {2, 144, 4096, 144, true}, {2, 145, 4096, 145, false},
        {16, 160, 3000, 80, true},  {16, 161, 3000, 80, false}, {16, 113, 3072, 80, false}, {2, 145, 3072, 80, false},
        {24, 1024, 1500, 16, true}, {24, 1025, 1500, 20, false}, {24, 1024, 1500, 15, false},
        {8, 400, 2048, 99, false},  {8, 400, 2047, 99, true},   {4, 128, 1366, 0, true},    {4, 129, 1366, 0, false},  {6, 48, 900, 0, true},
        {6, 49, 900, 0, false},     {7, 80, 900, 0, true},      {7, 81, 900, 1, false},     {7, 81, 900, 2, true},     {25, 112, 4096, 112, true},
        {8, 614, 511, 20, false},    {8, 614, 512, 20, true},    {8, 160, 300, 20, true},    {25, 113, 900, 30, false},  {17, 112, 900, 0, true},   {17, 113, 900, 0, false},  {64, 112, 900, 0, true},    {64, 113, 2000, 9, false},  {4, 402, 1200, 0, false},  {8, 802, 1500, 0, false},
    };
    for (const auto &c : at) {
        CHECK(update_all_gather_quarters(c.tiles * c.fill, c.tiles, c.whole, c.P, 0) == c.quarters);
        CHECK(update_all_gather_quarters(c.tiles * c.fill, c.tiles, c.whole, c.P, 4 * c.tiles) == c.quarters);
        CHECK(!update_all_gather_quarters(c.tiles * c.fill, c.tiles, c.whole, c.P, 4 * c.tiles - 1));
    }
    struct { int64_t P, elems, tiles, whole; bool splits; } const apart[] = {
        {4, 100000000, 24415, 24413, false}, {5, 831 * 4096, 836, 826, true},   {5, 830 * 4096, 835, 825, false},  {8, 519 * 4096, 527, 511, true},
        {8, 518 * 4096, 526, 510, false},    {16, 260 * 4096, 276, 244, true},  {16, 259 * 4096, 275, 243, false}, {24, 225 * 4096, 249, 201, true},
        {64, 225 * 4096, 288, 161, true},    {64, 224 * 4096, 287, 160, false}, {8, 5000000, 2008, 1000, false},   {12, 2200000, 745, 0, false},
        {12, 5000000, 1678, 0, true},        {8, 16000000, 6408, 3200, true},   {5, 5000000, 1505, 1000, true},    {32, 1000000, 365, 0, false},
        {8, 5000000, 1436, 0, true},         {6, 5000000, 1641, 600, true},     {8, 3750000, 1202, 450, true},     {48, 450000, 144, 80, false},
        {6, 3513000, 1092, 600, true},       {16, 1060000, 440, 150, false},    {12, 1870000, 741, 250, false},    {32, 2641000, 1108, 400, true},
    };
    for (const auto &c : apart) {
        CHECK(update_all_gather_splits(c.elems, c.tiles, c.whole, c.P, 0) == c.splits);
        CHECK(!update_all_gather_splits(c.elems, c.tiles, c.whole, c.P, c.tiles - 1));
    }
}

// Whole tiles of a run against its tiles one by one.
static void whole_tiles()
{
    for (int64_t begin : {0, 1, 5, 4095, 4096, 4097, 8192, 12287})
        for (int64_t count : {1, 2, 4090, 4095, 4096, 4097, 8191, 8192, 8193, 20000, 20480})
            for (int32_t layer : {-1, 3}) {
                const dear_run r{layer < 0 ? 0 : begin, 7, count, 0, layer, 0, 0, 0};
                int64_t n = 0;
                for (int64_t k = 0; k < tiles_of_run(r); ++k) n += layer >= 0 && tile_of_run(r, k).count == DEAR_TILE_ELEMS;
                CHECK(whole_tiles_of_run(r) == n);
            }
}

// dear_iteration in one launch: few replicas, or small calls and open tiles.
static void at_once()
{
    struct { int g; int64_t P, elems, tiles; bool gbar, once; } const at[] = {
        {4, 1, 1, 1, true, true},             {4, 2, 100000000, 24500, true, true},  {4, 3, 24999999, 6200, false, false}, {4, 3, 25000000, 6200, true, true},
        {4, 4, 39999999, 9800, false, false}, {4, 4, 40000000, 9800, false, true},   {4, 4, 40000000, 9800, true, false},  {4, 4, 64000000, 15700, true, true},
        {4, 7, 1200000, 293, false, true},    {4, 8, 740000, 181, true, true},       {4, 8, 875000, 214, false, false},
        {4, 8, 960000, 239, false, false},    {4, 8, 960000, 240, false, true},      {4, 8, 1000000, 258, true, true},      {4, 8, 1000000, 259, true, false},
        {4, 8, 1056000, 258, false, true},    {4, 9, 1000000, 250, false, false},    {4, 12, 80000, 24, false, true},      {4, 12, 70000, 23, true, false},
        {4, 13, 70000, 38, false, false},     {4, 16, 60000, 47, false, false},      {4, 16, 60000, 48, true, true},       {4, 64, 100000, 92, false, true},
        {4, 64, 100000, 91, true, false},     {4, 9, 5000, 10, true, true},          {4, 16, 1000000, 516, false, true},   {4, 32, 6000000, 2000, false, false},
        {4, 64, 468750, 246, false, false},   {4, 24, 468750, 246, false, true},     {4, 64, 300000, 246, false, true},      {4, 64, 1500000, 1064, true, true},
        {2, 2, 24999999, 6200, true, false},  {2, 2, 25000000, 6200, true, true},    {2, 4, 2900000, 710, false, true},    {2, 5, 1800000, 444, false, true},
        {2, 5, 2080000, 513, false, false},   {2, 4, 2300000, 566, true, false},     {2, 2, 2300000, 566, false, true},      {2, 6, 1916700, 474, true, true},     {2, 11, 1337000, 640, true, true},     {2, 5, 3950000, 1354, false, true},    {2, 8, 1708768, 473, true, true},     {2, 6, 2600000, 1006, false, false},
        {2, 5, 2300000, 566, false, false},   {2, 8, 1437500, 359, true, true},      {2, 8, 30000, 18, false, true},       {2, 9, 60000, 36, false, true},
        {2, 9, 60000, 35, false, false},      {2, 32, 100000, 124, true, true},      {2, 32, 100000, 123, false, false},   {2, 8, 2600000, 1006, true, false},
        {2, 8, 780000, 306, true, true},      {2, 8, 2000000, 1006, true, true},     {2, 8, 6000000, 3008, true, false},   {2, 8, 4500000, 3008, true, true},
        {2, 32, 600000, 330, false, true},    {2, 32, 2000000, 1030, false, false},  {2, 32, 1500000, 1030, false, true},  {2, 64, 300000, 330, false, true},    {2, 64, 300000, 152, true, false},
    };
    CHECK(iteration_at_once_residency(true, false, 1, 25000000, 6104) == 2 && iteration_at_once_residency(true, false, 1, 24999999, 6104) == 0);
    CHECK(iteration_at_once_residency(true, true, 1, 89000000, 21800) == 2 && iteration_at_once_residency(true, true, 1, 90000000, 22000) == 1);
    CHECK(iteration_at_once_residency(true, false, 1, 300000000, 73300) == 2 && iteration_at_once_residency(true, false, 2, 25000000, 6104) == 1);
    CHECK(iteration_at_once_residency(false, true, 1, 4000000, 980) == 2 && iteration_at_once_residency(false, true, 3, 3900000, 960) == 0);
    CHECK(iteration_at_once_residency(true, true, 2, 30000000, 12000) == 0);
    for (const auto &c : at) {
        CHECK(iteration_gathers_at_once(c.g, c.P, c.elems, c.tiles, c.gbar, 0) == c.once);
        CHECK(!iteration_gathers_at_once(c.g, c.P, c.elems, c.tiles, c.gbar, 1 << 20));
    }
}

// Tables of a context: each on 256 bytes, none over another, all within the allocation, whatever lies before them.
static void tables()
{
    for (bool sent : {true, false})
        for (int64_t runs : {1, 5, 7, 171, 1000})
            for (int64_t tiles : {runs, runs + 3, 40 * runs})
                for (int64_t L : {1, 3, 161})
                    for (int64_t P : {1, 7, 64}) {
                        const size_t places = L * 32, pointers = L * P * sizeof(void *);
                        const size_t room = (tiles + TILES_BEHIND) * sizeof(dear_tile);
                        const table_layout t = lay_out_tables(sent, tiles, runs, places, pointers);
                        CHECK(t.uploaded % 256 == 0 && t.places % 256 == 0 && t.grad % 256 == 0 && t.param % 256 == 0);
                        CHECK(sent ? t.uploaded == 0 && t.places >= room
                                   : t.uploaded >= room && t.places >= t.uploaded + runs * sizeof(dear_run));
                        CHECK(t.grad >= t.places + places && t.param >= t.grad + pointers && t.end == t.param + pointers);
                    }
}

int main()
{
    tables();
    grids();
    half_tiles();
    pairs_of_parts();
    iteration();
    whole_tiles();
    update_and_gather();
    at_once();
    std::printf("launch_rules: ok\n");
    return 0;
}
