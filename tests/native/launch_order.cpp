// Host-only check (dear_internal.h) of the all-gather's numbering -- for every replica, each part of a launch belongs to
// exactly one workgroup, in chunks and behind them, whatever the part count, in a grid that HIP and a bound allow -- and of the
// rule that takes a whole iteration in one launch: none that HIP would not take, none with a bounded grid.  Exits non-zero on the first mistake.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "dear_internal.h"

int main()
{
    const unsigned chunk = 4096;
    for (unsigned run : {0u, 1u})
        for (int64_t width : {0, 8, 28, 56, 256, 1000, 100000})
            for (int64_t P : {int64_t(1), int64_t(7), int64_t(64), int64_t(4095), int64_t(4096), int64_t(5000), MAX_GRID / 4})
                for (unsigned tiles : {1u, 2u, 3u, 4u, 5u, 511u, 1021u, 1023u, 1024u, 1025u, 1026u, 2047u, 2048u, 2049u}) {
                    const unsigned parts = tiles * AG_SPLIT;
                    if (!all_gather_fits(tiles, P, 0) || all_gather_bounded(tiles, P, width)) continue;
                    const unsigned whole = parts / chunk * chunk;
                    const all_gather_order o = all_gather_numbering(run, width, whole, parts, P);
                    std::vector<int> seen(parts, 0);
                    for (unsigned r = 0; r < whole + o.len; ++r) {
                        const unsigned first = r < whole ? r / chunk * chunk : whole;
                        const unsigned id = first + all_gather_part(r - first, o.run);
                        if (id < parts) ++seen[id];
                        if (id / AG_SPLIT >= tiles + TILES_BEHIND) seen[0] = 2;  // reads a tile that is not there
                    }
                    const int64_t grid = (whole + int64_t(o.len)) * P;
                    bool ok = grid <= MAX_GRID && (width == 0 || grid <= width);
                    for (int n : seen) ok = ok && n == 1;
                    if (!ok) {
                        std::fprintf(stderr, "FAILED run=%u width=%d P=%lld tiles=%u\n", run, int(width), (long long)P, tiles);
                        std::exit(1);
                    }
                }
    for (int g = 2; g <= 4; g += 2)
        for (int64_t P = 1; P <= 70; ++P)
            for (int64_t elems = 1; elems < int64_t(1) << 38; elems *= 3)
                for (int64_t tiles : {elems / DEAR_TILE_ELEMS + P, elems / 700 + P, MAX_GRID / AG_SPLIT, MAX_GRID / AG_SPLIT + 1}) {
                    bool ok = true;
                    for (bool gbar : {false, true}) {
                        const bool once = iteration_gathers_at_once(g, P, elems, tiles, gbar, 0);
                        ok = ok && !iteration_gathers_at_once(g, P, elems, tiles, gbar, 256) && (!once || tiles * AG_SPLIT <= MAX_GRID);
                        if (once && P > 4) ok = ok && P * (2 * elems - tiles * DEAR_TILE_ELEMS) <= 12000000;
                    }
                    if (!ok) {
                        std::fprintf(stderr, "FAILED at once g=%d P=%lld elems=%lld tiles=%lld\n", g, (long long)P, (long long)elems, (long long)tiles);
                        std::exit(1);
                    }
                }
    // a bound holds for the grid that dear_update_all_gather's one kernel gets
    for (int64_t width : {1, 5, 50, 64, 160, 256, 640, 641, 1000, 5000})
        for (int64_t tiles = 1; tiles < 1100; ++tiles)
            for (int64_t elems : {tiles, tiles * 700, tiles * 2100, tiles * DEAR_TILE_ELEMS}) {
                const bool bounded = tiles > width;
                const int64_t grid = bounded ? width : update_all_gather_quarters(elems, tiles, elems / DEAR_TILE_ELEMS, 8, width) ? tiles * 4 : tiles;
                if (grid > width) {
                    std::fprintf(stderr, "FAILED update + all-gather: %lld workgroups, bound %lld\n", (long long)grid, (long long)width);
                    std::exit(1);
                }
            }
    std::printf("launch_order: ok\n");
    return 0;
}
