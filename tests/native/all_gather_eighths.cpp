// Host-only check (dear_internal.h): where each XCD takes an eighth of a chunk, every part belongs to exactly one workgroup, in whole
// chunks and in last ones, and the rule takes no short launch and none of mostly empty tiles.  Exits non-zero on the first mistake.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "dear_internal.h"

int main()
{
    const unsigned chunk = 4096;
    for (unsigned tiles = 1; tiles < 5000; tiles += tiles < 40 ? 1 : 61)
        for (int64_t P : {int64_t(1), int64_t(24), int64_t(64)}) {
            const unsigned parts = tiles * AG_SPLIT, whole = parts / chunk * chunk;
            const all_gather_order o = all_gather_numbering(0, 0, whole, parts, P);
            if (o.len % 8) continue;
            std::vector<int> seen(parts, 0);
            for (unsigned r = 0; r < whole + o.len; ++r) {
                const unsigned first = r < whole ? r / chunk * chunk : whole;
                const unsigned id = first + all_gather_part_of_eighth(r - first, r < whole ? chunk : o.len);
                if (id < parts) ++seen[id];
                if (id / AG_SPLIT >= tiles + TILES_BEHIND) seen[0] = 2;  // reads a tile that is not there
            }
            for (int n : seen)
                if (n != 1) {
                    std::fprintf(stderr, "FAILED tiles=%u P=%lld\n", tiles, (long long)P);
                    return 1;
                }
        }
    for (int64_t P = 1; P < 100; ++P)
        for (int64_t tiles : {1, 900, 959, 960, 1599, 1600, 2047, 2048, 30000})
            if (all_gather_in_eighths(tiles * DEAR_TILE_ELEMS, tiles, P) != (tiles >= (P >= 24 ? 960 : P >= 12 ? 1600 : 2048) && (P >= 5 || tiles < 5000)) ||
                all_gather_in_eighths(tiles * DEAR_TILE_ELEMS / 2 - 1, tiles, P)) {
                std::fprintf(stderr, "FAILED rule tiles=%lld P=%lld\n", (long long)tiles, (long long)P);
                return 1;
            }
    std::printf("all_gather_eighths: ok\n");
    return 0;
}
