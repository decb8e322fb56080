// Internal definitions shared by the host planner and the HIP side of libdear.
#pragma once

#include <cstdint>
#include <vector>

#include "dear.h"

struct dear_plan_s {
    int32_t L = 0, B = 0, P = 0, g = 0;
    int64_t threshold_bytes = 0;
    int64_t N = 0;               // sum of layer sizes
    int64_t row_len = 0;         // sum of S_b: one worker's row of a shard buffer
    std::vector<int64_t> layer_sizes, layer_offset;
    std::vector<int32_t> layer_bucket;
    std::vector<int32_t> bucket_first_layer, bucket_n_layers;
    std::vector<int64_t> bucket_len, bucket_shard_len, bucket_shard_base;
};

typedef dear_tile_t dear_tile;
static_assert(sizeof(dear_tile) == 32, "tile descriptors are read as two 16-byte loads");

constexpr int DEAR_BLOCK = 256;  // threads per workgroup = 4 wavefronts

// ------------------------------------------------ which launches a call makes, by its sizes alone
//
// HIP takes fewer than 2^32 threads along a dimension of a launch: a grid has at most this many workgroups.
constexpr int64_t MAX_GRID = 0xffffffffu / DEAR_BLOCK;

constexpr int AG_SPLIT = DEAR_TILE_ELEMS / (4 * DEAR_BLOCK);  // all-gather: workgroups per tile and replica

inline bool all_gather_bounded(int64_t tiles, int64_t n_workers, int64_t max_workgroups)
{
    return max_workgroups > 0 && tiles * AG_SPLIT * n_workers > max_workgroups;
}

// The bounded form strides over whole tiles, so that its grid is small; its item count fits 31 bits.
inline bool all_gather_fits(int64_t tiles, int64_t n_workers, int64_t max_workgroups)
{
    const int64_t items = tiles * AG_SPLIT * n_workers;
    if (!all_gather_bounded(tiles, n_workers, max_workgroups)) return items <= MAX_GRID;
    return items <= 0x7fffffff && (max_workgroups <= MAX_GRID || tiles <= MAX_GRID);
}

// dear_update_all_gather as one kernel writes all P replicas from the workgroup that updated: P write streams at
// once, which HBM sustains worse the more there are (5.4 TB/s at P = 8, against 6.5 replica by replica).  From
// UAG_SPLIT_P replicas on the 4 bytes per element that one kernel saves are worth less than that, if the
// launch is long enough to pay for a second one: UAG_SPLIT_TILES tile copies are about 25 us.  us per iteration
// of reduce-scatters and these calls, one kernel / update, then all-gather: 100 M elements in 64 MB buckets
// P = 2 710 / 757, P = 3 857 / 878, P = 4 1016 / 1011; 25 M elements in 25 MB buckets P = 8 430 / 400;
// BERT-Base-shaped P = 16 3173 / 2826; 5 M elements in 4 MB buckets P = 8 115 / 131; 36 M elements P = 5 in one call
// 340 / 346, in 64 MB buckets 431 / 423, P = 6 474 / 463.  Beyond the largest all-gather the one kernel, whose
// grid is the tile count alone, still takes the call.
constexpr int64_t UAG_SPLIT_P = 6, UAG_SPLIT_TILES = 8192;

inline bool update_all_gather_splits(int64_t tiles, int64_t P, int64_t max_workgroups)
{
    const bool bounded = max_workgroups > 0 && tiles > max_workgroups;
    return !bounded && P >= UAG_SPLIT_P && tiles * P >= UAG_SPLIT_TILES && all_gather_fits(tiles, P, max_workgroups);
}

// Cuts every bucket of the plan into tiles (plan.cpp).
int64_t dear_emit_tiles(const dear_plan_s &pl, int32_t b_first, int32_t b_last, dear_tile *out,
                        int64_t capacity, int64_t *tile_begin);
void dear_build_tiles(const dear_plan_s &pl, std::vector<dear_tile> &tiles, std::vector<int64_t> &tile_begin);
