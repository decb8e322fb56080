// Host-only check (dear_internal.h) of the reduce-scatter's and the update's rows of items, each item to exactly one workgroup whatever their
// number, and of the rule for its shape: never more replicas in flight than there are, and only what there are kernels for.
// Exits non-zero on the first mistake.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "dear_internal.h"

int main()
{
    for (unsigned run : {0u, 4u, 6u, 9u})
        for (unsigned n = 1; n < (run < 9 ? 2100 : 12400); n += n < 1100 ? 1 : 37) {
            std::vector<int> seen(n, 0);
            for (unsigned b = 0; b < n; ++b) {
                const unsigned item = item_in_rows(b, run, n);
                if (item >= n || seen[item]++) {
                    std::fprintf(stderr, "FAILED run=%u n=%u b=%u item=%u\n", run, n, b, item);
                    return 1;
                }
            }
        }
    // one of the largest grids: the rows end where they do in small ones
    const unsigned most = static_cast<unsigned>(MAX_GRID), rest = most % (8u << 6);
    for (unsigned b = most - rest; b < most; ++b)
        if (item_in_rows(b, 6, most) != b) return 1;
    for (bool bf16 : {false, true})
        for (bool updates : {false, true})
            for (bool caches_w : {false, true})
                for (int64_t P = 1; P <= 130; ++P)
                    for (int64_t tiles : {1, 15, 16, 63, 64, 96, 127, 128, 191, 192, 255, 256, 319, 512, 1023, 1024, 2048, 4096, 5999, 6000, 30000})
                        for (int64_t percent : {1, 24, 39, 50, 79, 80, 100})
                            for (int64_t whole : {int64_t(0), tiles}) {
                                const reduce_scatter_shape s =
                                    reduce_scatter_shape_of(bf16, updates, caches_w, P, tiles * DEAR_TILE_ELEMS * percent / 100, tiles, whole);
                                const bool depth = s.depth == 0 || s.depth == 1 || s.depth == 2 || s.depth == 4 || s.depth == 8;
                                if (!depth || s.depth > P || s.residency < 0 || s.residency > 4 || s.residency == 1 || s.run < 0 || s.run > 6 ||
                                    (s.tiles && (s.depth == 0 || whole))) {
                                    std::fprintf(stderr, "FAILED bf16=%d updates=%d P=%lld tiles=%lld percent=%lld\n", bf16, updates,
                                                 (long long)P, (long long)tiles, (long long)percent);
                                    return 1;
                                }
                            }
    if (!pointer_table_fits(1, (int64_t{1} << 29) - 1) || pointer_table_fits(2, int64_t{1} << 28)) return 1;
    if (shard_update_run(1, 11999) != 0 || shard_update_run(1, 12000) != 9 || shard_update_run(1, MAX_GRID) != 9 || shard_update_run(2, 12000) != 0) return 1;
    std::printf("reduce_scatter_shapes: ok\n");
    return 0;
}
