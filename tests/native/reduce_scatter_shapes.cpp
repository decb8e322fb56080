// Host-only check (dear_internal.h) of the reduce-scatter's and the update's rows of items, each item to exactly one workgroup whatever their
// number, and of the rule for its shape: never more replicas in flight than there are, and only what there are kernels for (one in flight is
// for one replica).
// Exits non-zero on the first mistake.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "dear_internal.h"

// Asked for on stdin: bf16 updates caches_w P elems tiles long cut, a line each; answered with depth, residency, run, tiles.
static int answer()
{
    int bf16, updates, caches_w;
    long long P, elems, tiles, long_tiles, cut;
    while (std::scanf("%d %d %d %lld %lld %lld %lld %lld", &bf16, &updates, &caches_w, &P, &elems, &tiles, &long_tiles, &cut) == 8) {
        const reduce_scatter_shape s = reduce_scatter_shape_of(bf16, updates, caches_w, P, elems, tiles, long_tiles, cut);
        std::printf("%d %d %d %d\n", s.depth, s.residency, s.run, static_cast<int>(s.tiles));
    }
    return 0;
}

// Tiles of a run that begin or end inside a vector, or lie in more than one part, against its tiles one by one.
static bool counted_tiles()
{
    for (int64_t vector : {4, 8})
        for (int64_t begin : {0, 1, 4, 8, 3072, 4092, 4095, 4096, 12287})
            for (int64_t count : {1, 3, 4, 8, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 20000, 20004})
                for (int32_t layer : {-1, 3}) {
                    const dear_run r{layer < 0 ? 0 : begin, 7, count, 0, layer, 0, 0, 0};
                    int64_t n = 0, n_long = 0;
                    for (int64_t k = 0; k < tiles_of_run(r); ++k) {
                        const dear_tile t = tile_of_run(r, k);
                        n += layer >= 0 && (t.src_begin % vector != 0 || (t.src_begin + t.count) % vector != 0);
                        int64_t parts = 0;
                        for (int64_t first = t.src_begin / vector; first * vector < t.src_begin + t.count; first += DEAR_BLOCK) ++parts;
                        n_long += layer >= 0 && parts > 1;
                    }
                    if (cut_tiles_of_run(r, vector) != n || long_tiles_of_run(r, vector) != n_long) return false;
                }
    return true;
}

// Launches that the batch kernel keeps, and their neighbours that it does not: full tiles, nothing cut or all of them.
static bool batch_kernel()
{
    struct { bool bf16, updates; int64_t P, tiles; bool cut, batch; } const at[] = {
        // 25 MB buckets of a convolutional net, eight workers
        {false, true, 8, 585, false, true},  {false, true, 8, 1116, false, true}, {false, true, 8, 1605, false, true},
        {false, true, 8, 2047, false, true}, {false, true, 8, 2048, false, false}, {false, true, 8, 1116, true, false},
        {false, true, 9, 1116, false, false}, {false, false, 8, 159, false, true}, {false, false, 8, 160, false, false},
        {false, false, 3, 2047, false, true}, {false, false, 4, 1116, false, false}, {false, true, 12, 64, false, true},
        {false, true, 12, 63, false, false}, {false, true, 64, 159, false, true}, {false, true, 64, 160, false, false},
        {false, false, 12, 100, false, false}, {false, false, 20, 100, false, true}, {false, false, 7, 159, true, true},
        {false, false, 7, 160, true, false}, {true, true, 8, 2047, false, true}, {true, true, 16, 699, false, true},
        {true, true, 16, 700, false, false}, {true, true, 24, 131, false, false}, {true, true, 24, 132, false, true},
        {true, true, 24, 287, false, true},  {true, true, 24, 288, false, false}, {true, false, 24, 159, false, true},
        {true, false, 24, 160, false, false}, {true, true, 8, 109, true, false}, {true, true, 8, 299, true, true},
        {true, true, 8, 300, true, false},   {true, false, 4, 159, true, true}, {true, false, 4, 160, true, false},
        {true, true, 4, 110, false, true},   {true, true, 4, 1116, false, false}, {true, true, 1, 127, false, false},
        {true, true, 2, 128, false, true},   {true, true, 2, 700, false, false}, {true, true, 2, 200, true, false},
        {true, true, 6, 899, false, true},   {true, true, 6, 900, false, false}, {true, true, 8, 900, false, true},
        {true, true, 3, 400, true, false},   {true, false, 2, 400, true, false}, {true, false, 2, 2047, false, true},
    };
    for (const auto &c : at) {
        const int64_t elems = c.tiles * DEAR_TILE_ELEMS, cut = c.cut ? (c.tiles + 7) / 8 : (c.tiles - 1) / 8;
        if ((reduce_scatter_shape_of(c.bf16, c.updates, false, c.P, elems, c.tiles, c.tiles, cut).depth == 0) != c.batch) {
            std::fprintf(stderr, "FAILED batch kernel: bf16=%d updates=%d P=%lld tiles=%lld cut=%d\n", c.bf16, c.updates, (long long)c.P,
                         (long long)c.tiles, c.cut);
            return false;
        }
    }
    return true;
}

int main(int argc, char **)
{
    if (argc > 1) return answer();
    if (!counted_tiles() || !batch_kernel()) return 1;
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
                        for (int64_t percent : {1, 24, 39, 50, 79, 80, 87, 100})
                            for (int64_t long_tiles : {int64_t(0), tiles / 12, tiles}) {
                                const int64_t cut = percent % 2 ? tiles : 0;
                                const reduce_scatter_shape s = reduce_scatter_shape_of(
                                    bf16, updates, caches_w, P, tiles * DEAR_TILE_ELEMS * percent / 100, tiles, long_tiles, cut);
                                const bool depth = s.depth == 0 || s.depth == 1 || s.depth == 2 || s.depth == 4 || s.depth == 8;
                                if (!depth || s.depth > P || (s.depth == 1 && P > 1) || s.residency < 0 || s.residency > 4 || s.residency == 1 || s.run < 0 || s.run > 6 ||
                                    (s.tiles && (s.depth == 0 || long_tiles == tiles))) {
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
