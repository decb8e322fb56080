// Internal definitions shared by the host planner and the HIP side of libdear.
#pragma once

#include <cstdint>
#include <vector>

#include "dear.h"

#ifdef __HIPCC__
#define DEAR_HOST_DEVICE __host__ __device__
#else
#define DEAR_HOST_DEVICE
#endif

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

// A run: `count` elements of one layer within one shard, or padding slots of one shard (layer -1, src_begin 0).  The tile
// table follows from the runs.  Where they are a few hundred and the tiles thousands, it is the runs that are uploaded, and a kernel
// cuts them (expand_runs_kernel); small tables are cut on the host and uploaded as they are.
struct dear_run {
    int64_t src_begin, dst_begin, count;
    int64_t first_tile;  // its tiles' place in the table
    int32_t layer, shard, bucket, reserved;
};

DEAR_HOST_DEVICE inline int64_t tiles_of_run(const dear_run &r)
{
    return (r.src_begin + r.count + DEAR_TILE_ELEMS - 1) / DEAR_TILE_ELEMS - r.src_begin / DEAR_TILE_ELEMS;
}

// Those of its tiles that are whole ones of a layer.
inline int64_t whole_tiles_of_run(const dear_run &r)
{
    const int64_t n = (r.src_begin + r.count) / DEAR_TILE_ELEMS - (r.src_begin + DEAR_TILE_ELEMS - 1) / DEAR_TILE_ELEMS;
    return r.layer < 0 || n < 0 ? 0 : n;
}

// Those of its tiles that begin or end inside a 16-byte vector of `vector` gradients, 4 or 8: masks, as a static call counts hundreds
// of runs and does not know the type when it is compiled.
inline int64_t cut_tiles_of_run(const dear_run &r, int64_t vector)
{
    if (r.layer < 0) return 0;
    const bool begins = (r.src_begin & (vector - 1)) != 0, ends = ((r.src_begin + r.count) & (vector - 1)) != 0;
    return tiles_of_run(r) > 1 ? begins + ends : begins || ends;
}

DEAR_HOST_DEVICE inline dear_tile tile_of_run(const dear_run &r, int64_t k)
{
    const int64_t cut = (r.src_begin / DEAR_TILE_ELEMS + k) * DEAR_TILE_ELEMS, end = r.src_begin + r.count;
    const int64_t lo = k == 0 ? r.src_begin : cut, hi = cut + DEAR_TILE_ELEMS < end ? cut + DEAR_TILE_ELEMS : end;
    return {r.layer < 0 ? 0 : lo, r.dst_begin + (lo - r.src_begin), static_cast<int32_t>(hi - lo), r.layer, r.shard, r.bucket};
}

constexpr int DEAR_BLOCK = 256;  // threads per workgroup = 4 wavefronts

// Those of its tiles that lie in more than one part of the reduce-scatter, DEAR_BLOCK vectors of `vector` gradients.
inline int64_t long_tiles_of_run(const dear_run &r, int64_t vector)
{
    if (r.layer < 0) return 0;
    const int64_t n = tiles_of_run(r);
    auto is_long = [&](int64_t k) {
        const dear_tile t = tile_of_run(r, k);
        return ((t.src_begin + t.count - 1) & -vector) - (t.src_begin & -vector) >= DEAR_BLOCK * vector;
    };
    return n > 1 ? n - 2 + is_long(0) + is_long(n - 1) : is_long(0);
}

// What the device's copy of a tile carries in the place of its bucket, for the all-gather.
constexpr int TILE_FIRST = 1, TILE_LAST = 2;  // of its run: the tiles of one layer and shard
constexpr int TILE_OWN_SHIFT = 4;             // the replicas' tensors lie differently: each has a shift of its own
constexpr int TILE_SHIFT_BIT = 8;             // the replicas' common shift from this bit on

// Elements between the last 128-byte line that begins at or before p, and p (16-byte aligned).
DEAR_HOST_DEVICE inline int line_shift(uintptr_t p) { return static_cast<int>((p >> 2) & 31); }

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

// Whether some of a launch's tiles are whole.  Weights between short vectors give whole tiles and nearly empty ones, tensors
// that are all shorter than a tile none; elements and tiles alone do not tell one from the other.
inline bool some_whole(int64_t whole, int64_t tiles) { return whole * 64 >= tiles; }

// The batch kernel of the bf16 reduce-scatter takes half a tile a workgroup (one 16-byte vector a lane instead of two) where a launch
// is so short that whole tiles leave CUs idle, unless its tensors are all so short that most second halves are empty.  GPU time, us,
// whole tiles / halves: reduce-scatter alone P = 8 0.2 M elements 4.47 / 4.06, 0.4 M 4.83 / 4.38, 0.8 M 5.39 / 5.41,
// 1.6 M 7.32 / 7.71; P = 32 0.4 M 11.9 / 10.8, 1.6 M 21.6 / 22.5.  With the update the line lies further out, behind an all-gather
// that follows at once or later: all reduce-scatters + updates, then all all-gathers of up to eight buckets of 150 / 300 / 550 / 850
// tiles, change in %: P = 4 -2 / -5 / -5 / -1, P = 8 -5 / -6 / -5 / -3, P = 16 -3 / -6 / -4 / -3, P = 32 -9 / -5 / +1 / -3, P = 48
// -7 / -3 / +5 / +2, P = 64 -7 / -7 / +4 / +1; iteration of one bucket P = 4 0 / -5 / -3 / +1, P = 8 -5 / -7 / -7 / -2, P = 32
// -12 / -6 / -7 / -2, P = 64 -8 / -4 / -4 / -3; one bucket of weights and short vectors, 15 to 90 % full, P = 3 to 64, 80 to 850 tiles
// -18 to +1.
// Short tensors, iteration in two launches: P = 9 60 of 400 elements 8.20 / 8.62, of 1000 8.90 / 9.33, of 1600 9.85 / 9.08;
// P = 32 of 1000 17.7 / 18.5, of 1600 20.2 / 18.3; P = 64 of 1000 35.2 / 37.5, of 1600 35.6 / 38.4, of 2400 42.9 / 38.5.
// Reduce-scatter + update P = 10 396 tensors of 1430 9.33 / 10.08; in a dozen tiles empty halves cost nothing (P = 8 2460 elements in
// 5 tensors 5.96 / 5.64).
inline bool half_tiles_filled(int64_t elems, int64_t tiles, int64_t whole)
{
    return tiles <= 16 || some_whole(whole, tiles) || elems >= tiles * (tiles <= 200 ? 1024 : 1536);
}

inline bool reduce_scatter_half_tiles(bool updates, int64_t max_workgroups, int64_t elems, int64_t tiles, int64_t whole)
{
    return max_workgroups == 0 && tiles <= (updates ? 1024 : 160) && half_tiles_filled(elems, tiles, whole);
}

// How the unbounded all-gather numbers its workgroups (see all_gather_kernel).  Where HIP would not take a launch with a
// rounded last chunk, or a bound on the grid would not allow it, that chunk stays as it falls.
struct all_gather_order {
    unsigned len, run;
};

// Room behind a context's tile table: the workgroups of a rounded last chunk read up to 15 parts beyond the last.
constexpr int TILES_BEHIND = 4;

// Offsets of a context's device tables in their one allocation: tiles first; from `uploaded` on, what the host sends (the
// tiles, or the runs that a kernel cuts into them); layer places, gradient and parameter pointers; `end` bytes in all.
// Every table starts on a multiple of 256 bytes.  Packed behind the runs, of 48 bytes each, the pointer tables started anywhere on
// 16 bytes: ResNet-50, P = 8 fp32, a bucket at a time, us per iteration packed / aligned 355.2 / 354.5, 357.7 / 356.7 and
// 354.1 / 353.5 (spread 0.1).
struct table_layout {
    size_t uploaded, places, grad, param, end;
};

inline table_layout lay_out_tables(bool tiles_sent, int64_t n_tiles, int64_t n_runs, size_t place_bytes, size_t pointer_bytes)
{
    auto aligned = [](size_t n) { return (n + 255) & ~size_t(255); };
    const size_t tiles = aligned((n_tiles + TILES_BEHIND) * sizeof(dear_tile));
    table_layout t{};
    t.uploaded = tiles_sent ? 0 : tiles;
    t.places = tiles_sent ? tiles : tiles + aligned(n_runs * sizeof(dear_run));
    t.grad = t.places + aligned(place_bytes);
    t.param = t.grad + aligned(pointer_bytes);
    t.end = t.param + pointer_bytes;
    return t;
}

// Part of a chunk that a replica's r-th workgroup takes: XCD r % 8 takes 2^run parts in a row out of every 8 * 2^run.
DEAR_HOST_DEVICE inline unsigned all_gather_part(unsigned r, unsigned run)
{
    return (r & ~((8u << run) - 1)) | (r & 7) << run | (r >> 3 & ((1u << run) - 1));
}

// The same where every XCD takes an eighth of the chunk, its parts in a row: len, the chunk's workgroups per replica, is a
// multiple of 8.
DEAR_HOST_DEVICE inline unsigned all_gather_part_of_eighth(unsigned r, unsigned len) { return (r & 7) * (len >> 3) + (r >> 3); }

// Where it is: an XCD then writes 2 MiB of a replica in a row and not every eighth 4 KiB, and of the lines that two
// workgroups write in halves, at the ends of runs, both halves go through one L2.  Each next part = 1, the all-gather alone / a pass
// of reduce-scatter with update and all-gather / dear_iteration, sets of buffers in turn, 20 ragged tensors: fp32 P = 4 2300 tiles
// 0.94 / 0.99 / 0.99  4500 0.97 / 0.98 / 0.99, P = 8 2300 0.98 / 0.99 / 1.00  4500 0.99 / 1.00 / 0.99, P = 16 3000 0.97 / 0.99 / 0.99,
// P = 32 900 0.91 / 0.96 / 0.96  1800 0.93 / 0.97 / 0.97  3000 0.95 / 0.98 / 0.97, bf16 P = 16 2300 0.97 / 0.98 / 0.98, P = 64 900
// 0.93 / 0.94 / 0.94  1800 0.89 / 0.93 / 0.92; ResNet-50-shaped P = 64 0.95 / 0.95 / 0.95, in one launch 0.91 (6200 -> 6830 GB/s),
// BERT-Base-shaped P = 16 0.96 / 0.99 / 0.99, in one launch 0.94.  One tensor, whose runs share no lines, gains nothing (P = 16 to 32
// 2000 to 5000 tiles 1.01 to 1.03).  2^run parts in a row (all_gather_part) cost 1-16 % up to run = 5, and 8 is level with eighths.
// Not below 2048 tiles, 32 MiB of w, whose values are read in the L2 of the XCD that wrote them, where each takes every eighth part:
// the same state over and over fp32 P = 4 900 tiles dear_iteration 1.17, 1800 1.03, P = 8 900 1.10, 1300 1.03, 1800 1.00 (with update
// in calls of their own 1.10, 1.08, 1.05), bf16 P = 8 900 1.19; with more replicas that weighs less: P = 12 1300 1.03, 1800 0.99,
// P = 16 1300 1.01, 1800 0.99, P = 32 900 0.94, bf16 1.02, 1300 0.99.
// Nor with many parts that short tensors leave empty, which give the XCDs unlike eighths: tensors of 900 elements, alone, P = 16 and
// 64, 2250 tiles 1.04 and 1.06; weights with short vectors between them, 80 % full, P = 8 2050 / 2600 / 3300 / 5200 tiles
// 1.04 / 1.03 / 1.04 / 1.03, P = 16 1.06 / 1.07 / 1.05 / 1.06, P = 24 1100 1.08, P = 64 960 / 2100 / 5300 1.07 / 1.07 / 1.07, though
// 6500 0.97, 0.93, - and 1.00.
// Few replicas lose a little in long launches (alone, P = 4 9000 1.01), one and two in most (P = 1 2600 to 4000 1.03, P = 2 7800 1.04
// to 1.05).
// Nor where the parts do not end at the same lines in all replicas (dear_ctx_s::replicas_alike): ResNet-50-shaped P = 64, replicas at
// multiples of 16 bytes that are none of 128 from one another 1.08, alike 0.94; 604 tensors on 16-byte boundaries P = 7
// 1.01 / 1.00 / 1.00, on lines 0.98 / 0.96 / 0.97.
inline bool all_gather_in_eighths(int64_t elems, int64_t tiles, int64_t n_workers)
{
    if (elems * 8 < tiles * DEAR_TILE_ELEMS * (tiles < 6000 ? 7 : 4)) return false;
    if (n_workers < 3 || tiles < (n_workers >= 24 ? 960 : n_workers >= 12 ? 1600 : 2048)) return false;
    return n_workers >= 5 || tiles < 5000;
}

inline all_gather_order all_gather_numbering(unsigned run, int64_t max_workgroups, unsigned whole, unsigned parts, int64_t n_workers)
{
    const unsigned last = parts - whole;
    const unsigned rounded = (last + (8u << run) - 1) & ~((8u << run) - 1);
    const int64_t most = max_workgroups > 0 && max_workgroups < MAX_GRID ? max_workgroups : MAX_GRID;
    if ((static_cast<int64_t>(whole) + rounded) * n_workers > most) return {last, 0};
    return {rounded, run};
}

// dear_update_all_gather as one kernel writes all P replicas from the workgroup that updated: P write streams at
// once, which HBM sustains worse the more there are (5.4 TB/s at P = 8, against 6.5 replica by replica).  From
// UAG_SPLIT_P replicas on the 4 bytes per element that one kernel saves are worth less than that, if the launch is long enough
// to pay for a second one and for the all-gather's workgroups for the parts of tiles that short tensors leave open (`open`
// elements), which cost as much as others.  GPU time of some buckets of one size, all reduce-scatters, then these calls, us, one
// kernel / two:
//   one tensor a bucket  P = 4 2.3 M elements 211 / 216  9 M 169 / 168   P = 5 1.8 M 193 / 202  2.8 M 175.7 / 175.9  3.4 M 171 / 164
//                        7.2 M 160 / 154
//                        P = 8 1.6 M 171 / 169  1.75 M 152 / 153  2.1 M 149 / 145 (2 of 12 buckets, the others smaller, 251 / 257)
//                        4.5 M 142 / 135
//                        P = 12 0.9 M 153 / 166  1.3 M 161 / 153  (in 76 tensors 1.6 M 32.8 / 33.9)
//                        P = 16 0.8 M 140 / 150  1 M 150 / 149  1.1 M 133 / 126  2.3 M 127 / 114
//                        P = 32 0.9 M 89 / 92  1 M 105 / 99   P = 64 0.7 M 63 / 67  0.9 M 79 / 80  1 M 96 / 89
//   tensors of 3500      P = 5 2.2 M 28.8 / 31.8  5 M 63.1 / 61.8   P = 8 2.2 M 38.6 / 40.7  5 M 86.2 / 82.0
//                        P = 16 1 M 31.8 / 33.6  5 M 149 / 135
//   tensors of 5000 (61 % full)  P = 8 2.2 M 45.4 / 46.6  5 M 90.5 / 97.8  16 M 294 / 299   P = 16 2.2 M 73 / 78
//                                P = 32 2.2 M 131 / 141
//   tensors of 3000 (73 %)       P = 5 5 M 62.1 / 64.9   P = 8 2.2 M 37.7 / 43.1  16 M 267 / 261
//                                P = 12 2.2 M 50.8 / 56.3  5 M 117 / 114   P = 32 1 M 56 / 61
//   tensors of 2400-9400 (74 %)  P = 6 5 M 76.4 / 72.0   P = 8 3.8 M 69.0 / 66.0
//   weights and short vectors    P = 6 3.5 M (78 %) 53.8 / 49.6   P = 8 2.5 M (89 %) 44.6 / 42.2  2.6 M (58 %) 53.0 / 51.9
//                                P = 12 1.9 M (62 %) 50.3 / 52.4   P = 16 1.1 M (59 %) 36.5 / 40.9   P = 32 2.6 M (58 %) 133 / 125
//   tensors of 2500 (61 %)       P = 5 16 M 195 / 211   P = 8 16 M 273 / 293   P = 32 2.2 M 129 / 143
// Beyond the largest all-gather the one kernel, whose grid is the tile count alone, still takes the call.
constexpr int64_t UAG_SPLIT_P = 5;

inline bool update_all_gather_splits(int64_t elems, int64_t tiles, int64_t whole, int64_t P, int64_t max_workgroups)
{
    constexpr int64_t M = 1000000;
    const bool bounded = max_workgroups > 0 && tiles > max_workgroups;
    const int64_t open = tiles * DEAR_TILE_ELEMS - elems;
    if (bounded || P < UAG_SPLIT_P || !all_gather_fits(tiles, P, max_workgroups)) return false;
    if (elems < (P > 16 ? 920000 : 17 * M / P)) return false;
    return some_whole(whole, tiles) ? (elems - open) * P >= 15 * M : (2 * elems - 3 * open) * P >= 24 * M;
}

// The one kernel in quarters of tiles, one vector a lane: where whole ones leave CUs idle, or keep them waiting for the few that
// hold most.  The more workgroups there are already, and the less all tiles hold, the more their number costs; it stays within a
// bound on the grid.  GPU time, all reduce-scatters, then these calls, us, whole tiles / quarters:
//   one bucket of weights and short vectors, by tiles a bucket
//     P = 2  113 7.6 / 6.5  199 8.0 / 7.4  357 10.7 / 8.9  586 11.7 / 11.1   P = 3 sixteen buckets of 166 (90 % full) 162 / 171
//     P = 8  91 9.7 / 9.0  128 9.8 / 9.0  182 9.9 / 9.4  297 16.2 / 14.5  466 15.6 / 13.9  614 (a tenth full) 11.1 / 12.9
//     P = 16 125 13.6 / 12.8  165 14.2 / 13.3  288 16.0 / 15.7  440 (60 % full) 36.5 / 37.9   P = 24 322 28.8 / 26.1  660 54.0 / 51.5
//     P = 32 106 19.9 / 18.2  138 22.5 / 23.6  238 24.1 / 26.3   P = 48 87 (eleven buckets) 283 / 259  132 28.9 / 30.0
//     P = 64 83 (nearly empty) 20.7 / 19.2  120 (two buckets) 65.8 / 66.7  138 37.4 / 43.1
//   eight buckets (fewer from P = 32 on) of one tensor
//     P = 2  24 tiles 47.5 / 39.7  64 51.7 / 50.7  110 59.0 / 57.8  150 63.4 / 65.3   P = 4  24 52.8 / 43.8  110 68.6 / 69.3
//            150 74.6 / 78.9
//     P = 8  24 62.6 / 51.5  110 84.0 / 84.8  150 99.0 / 101.1   P = 16 24 85.5 / 68.7  150 155.2 / 157.2
//     P = 32 24 127 / 103  110 221 / 233   P = 64 24 193 / 189  64 246 / 252  97 109 / 111
//   of tensors of one length
//     3000   P = 4 64 61.1 / 52.1  128 68.9 / 66.3   P = 16 64 96 / 82  128 107 / 106  143 123 / 126
//     900    P = 2 32 47.4 / 47.3  64 49.5 / 50.7   P = 8 56 60.8 / 60.0  72 65.4 / 65.7   P = 16 80 93.1 / 93.7  96 100 / 105
//            P = 24 104 141 / 132
//     beyond P = 2 800 of 1200 13.3 / 17.7   P = 8 400 of 1200 15.6 / 19.3  800 24.9 / 32.8
inline bool update_all_gather_quarters(int64_t elems, int64_t tiles, int64_t whole, int64_t P, int64_t max_workgroups)
{
    if (max_workgroups > 0 && tiles * 4 > max_workgroups) return false;
    if (P > 24) return tiles <= 112;
    const int64_t room = tiles * DEAR_TILE_ELEMS;
    if (!some_whole(whole, tiles)) return tiles <= (elems * 3 >= room ? 128 : P <= 6 ? 48 : P <= 16 ? 80 : 112);
    if (elems * 4 >= room * 3) return tiles <= (P <= 2 ? 144 : 112);
    return tiles <= (elems * 2 < room && elems * 8 >= room ? 1024 : 160);
}

// Cuts every bucket of the plan into runs and tiles (plan.cpp).
int64_t dear_emit_runs(const dear_plan_s &pl, int32_t b_first, int32_t b_last, dear_run *out, int64_t capacity,
                       int64_t *n_tiles, int64_t *tile_begin);
int64_t dear_emit_tiles(const dear_plan_s &pl, int32_t b_first, int32_t b_last, dear_tile *out,
                        int64_t capacity, int64_t *tile_begin);
void dear_build_tiles(const dear_plan_s &pl, std::vector<dear_tile> &tiles, std::vector<int64_t> &tile_begin);

// Writes into every run's bucket field what the all-gather wants to know about its tiles.  True: nearly all elements
// (seven eighths) are in runs whose cuts are lines in every replica, at the same elements (all_gather_in_eighths).
bool dear_mark_runs(const dear_plan_s &pl, float *const *param_ptrs, dear_run *runs, int64_t n_runs);

// Parts of a tile in the reduce-scatter: one 16-byte vector a lane.
inline int64_t reduce_scatter_split(bool bf16) { return DEAR_TILE_ELEMS / ((bf16 ? 8 : 4) * DEAR_BLOCK); }

// Item that the workgroup of index b takes, in the reduce-scatter and the update: XCD b % 8 takes 2^run items in a row out of every 8
// * 2^run, and what does not fill such a group goes as it falls.
DEAR_HOST_DEVICE inline unsigned item_in_rows(unsigned b, unsigned run, unsigned n_items)
{
    const unsigned group = 8u << run, first = b & ~(group - 1);
    if (n_items - first < group) return b;
    return first | (b & 7) << run | (b >> 3 & ((1u << run) - 1));
}

// The update's logarithm of the number of items (blocks of 1024 elements) in a row on an XCD: 2 MiB of each stream.  As they fall =
// 1, 64 / 256 / 512 / 1024 / 4096 in a row, sets of buffers in turn, the update alone: 336 M elements 1.03 /
// 0.95 / 0.96 / 0.97 / 0.97, 110 M 0.94 / 0.93 / 0.93 / 0.96 / 0.99, 64 M 0.95 / 0.94 / 0.92 / 0.97 / 1.03, 32 M
// 0.94 / 0.95 / 0.94 / 1.01 / 1.00, 25 M 0.99 / 0.96 / 0.95 / 1.03 / 1.00.  Pass of the three phases, 512: bf16 P = 8 336 M and 32 M
// 0.99, P = 16 110 M 0.99, P = 4 64 M 0.97, P = 64 25 M 1.00; one state over and over 0.99 / 1.00 / 0.99 / 0.98 / 1.00.  Shorter
// launches lie within 2 % either way (12 M 1.00 with 512, 8 M 1.00 with 256, one state over and over 1.02; 3 M 1.01 and 1.02) and keep
// their order.
// So do launches over some of the buckets, where every worker's row begins at a place of its own: 16 rows of BERT-Base-shaped buckets
// 6560 GB/s as they fall, 6337 with 512, 8 rows of BERT-Large-shaped ones 6315 and 6247.
inline unsigned shard_update_run(int64_t rows, int64_t n_items) { return rows > 1 || n_items < 12000 ? 0 : 9; }

// How an unbounded reduce-scatter goes: replicas in flight per lane (0: the batch kernel), workgroups that may share a CU (0: as
// many as fit), the logarithm of the number of items in a row on an XCD, and whether a workgroup takes whole tiles.
struct reduce_scatter_shape {
    int depth, residency, run;
    bool tiles;
};

// Where the batch kernel is the faster one still, below 2048 tiles: reduce_scatter_kernel gains by loads that never drain, and by
// taking the elements of vectors that a run cuts (`cut`: an eighth of the tiles begin or end inside one) along with the vectors, where
// the batch kernel has a pass of its own for them.  With up to eight replicas all loads of a workgroup are in flight at once anyway,
// so with nothing cut there is nothing to gain, and with the update w and v are loads that never stop beside them.  Seven
// replicas are two rounds of loads instead of one.  A launch that fills the chip less than once, and not by far, likes fewer, longer
// workgroups.  4256 launches (P = 1 to 64, 20 to 2000 tiles; one tensor, five, ragged lists, weights with short vectors between them;
// buffers in turn, cold), batch kernel = 1, mean (worst) of what would go instead:
//   nothing cut, up to eight replicas
//     fp32 with update  P = 3 1.02 (1.14)  5 1.02 (1.10)  6 1.01 (1.11)  7 1.03 (1.21)  8 1.02 (1.10), above 160 tiles 1.00
//     bf16 with update  P = 3 1.05 (1.18)  5, 6 and 7 1.02 (1.25)  8 1.01 (1.12)  1 and 2 0.97, but from 128 to 700 tiles 1.02 (1.07)
//     fp32 without      P = 3 1.04 (1.12)  4 to 8 below 160 tiles 1.04 (1.24), above 0.98
//     bf16 without      P = 2 1.01 (1.13)  3 to 8 below 160 tiles 1.07 (1.24), above 0.94
//   nothing cut, more
//     fp32, 64 to 160 tiles  with update P >= 12 1.06 (1.38)   without P = 9 to 16 0.94  P >= 24 1.08 (1.39)
//     bf16 with update       P = 12 and 16 below 700 tiles 1.02 (1.13)   P >= 24 from 132 to 288 1.04 (1.16)
//     bf16 without           P = 12 and 16 below 130 tiles 1.00 (1.09)   P >= 24 from 132 to 160 1.02 (1.14)
//   cut
//     fp32                   P <= 8 below 160 tiles 0.97, but 7 1.02 (1.07)   from 9 on 0.84
//     bf16                   from 9 on 0.82   P = 4 without update below 160 tiles 1.09   P = 7 below 160 1.04 (1.09)
//     bf16 with update       P = 5 to 7 from 40 to 300 tiles 1.05   P = 4 and 8 from 110 to 300 1.01
inline bool batch_kernel_stays(bool bf16, bool updates, int64_t P, int64_t tiles, bool cut)
{
    if (tiles >= 2048) return false;
    if (P == 7 && tiles < 160) return true;
    if (bf16 && updates && P <= 2) return !cut && tiles >= 128 && tiles < 700;
    if (cut || (bf16 && updates && P == 4)) {
        if (!bf16 || P < 4 || P > 8) return false;
        return updates ? tiles >= (P % 4 ? 40 : 110) && tiles < 300 : P == 4 && tiles < 160;
    }
    if (bf16 && updates && P >= 5 && P <= 7) return tiles < 900;
    if (P <= 8) return updates || P <= (bf16 ? 2 : 3) || tiles < 160;
    if (!bf16) return P >= (updates ? 12 : 20) && tiles >= 64 && tiles < 160;
    if (P < 24) return updates ? tiles < 700 : P >= 12 && tiles < 130;
    return tiles >= 132 && tiles < (updates ? 288 : 160);
}

// HBM serves P streams at once best with 24 to 48 KiB of loads in flight per CU, as long as they never stop: D loads of 4 KiB for
// each of the workgroups that share a CU, so 2/3 24 KiB, 2/4 32 in bf16 and 40 in fp32 (whose `residency` 4 lets five in), 4/2 32,
// 4/3 48, and with the update those of w and v beside them.  With more the streams get into each other's way, with fewer the
// latency shows; a launch that does not fill the chip wants more per workgroup.  So two replicas a lane and three or
// four workgroups a CU in long launches, four or eight replicas in short ones.  Depth / workgroups a CU (- as many as fit, r in rows),
// batch kernel = 1, means over the four kinds of lists, by tiles (the launches of batch_kernel_stays, and 1266 longer ones):
//   fp32 without update, 8/- | 4/- | 2/-
//     P = 9   20-45  0.81 | 0.88 | 1.07   46-63 0.80 | 0.85 | 1.03    64-90   0.84 | 0.83 | 0.97   128-170 0.90 | 0.89 | 0.90
//     P = 16  46-63  0.84 | 0.94 | 1.26   64-90 0.95 | 0.91 | 1.16    91-127  0.99 | 0.94 | 1.13   128-170 0.95 | 0.94 | 0.91
//     P = 32  46-63  0.77 | 0.93 | 1.36   64-90 0.93 | 0.91 | 1.22    91-127  0.99 | 0.94 | 1.21   128-170 0.98 | 0.97 | 0.96
//   4/- | 2/- | 2/4
//     320-1100  P = 4  1.00 | 1.00 | 1.06   P = 5  0.98 | 1.00 | 1.07   P = 6  0.99 | 0.99 | 1.03   P = 7  0.99 | 1.00 | 1.05
//               P = 8  0.98 | 1.00 | 1.02   395-480  P = 16 0.99 | 1.05 | 0.98   P = 24 0.99 | 1.04 | 0.96   P = 64 1.00 | 1.05 | 0.94
//   2/4r | 2/3r | 2/-r | 4/2
//     3000-5900  P = 4 0.99 | 1.03 | 0.98 | 1.13   P = 6 0.95 | 0.97 | 0.98 | 1.06   P = 8 0.94 | 0.96 | 0.98 | 0.99
//                P = 12 0.94 | 0.97 | 1.01 | 0.98   P = 16 0.96 | 0.98 | 1.02 | 0.99
//     24000 and more (one tensor, ragged, BERT-Base-shaped)  P = 8 1.02 | 0.99 | - | 0.98   P = 12 1.02 | 1.01 | - | 1.01
//                P = 16 1.03 | 1.02 | - | 0.99
//   fp32 with update, the same
//     3000-13000 P = 4 0.96 | 0.96 | 0.98 | 1.00   P = 6 0.96 | 0.95 | 1.00 | 1.01   P = 8 0.98 | 0.96 | 1.02 | 1.00
//                P = 12 0.99 | 0.98 | 1.05 | 1.02   P = 16 0.98 | 0.96 | 1.04 | 0.99
//     24000 and more  P = 8 1.03 | 0.99 | - | 1.00, dear_iteration 1.03 | 1.00 | - | 1.00
//   bf16 without, 8/- | 4/- | 2/-
//     P = 16  80-109 0.93 | 1.00 | 1.31   110-131 0.94 | 0.94 | 1.21   161-287 0.91 | 0.87 | 1.00   288-400 0.96 | 0.95 | 0.91
//     P = 24  80-109 0.85 | 0.94 | 1.30   110-131 0.86 | 0.93 | 1.27   132-160 0.97 | 0.92 | 1.21   161-287 0.86 | 0.82 | 0.98
//     P = 64  80-109 0.70 | 0.92 | 1.45   110-131 0.71 | 0.88 | 1.36   132-160 0.91 | 0.92 | 1.33   161-287 0.81 | 0.77 | 1.03
//   4/- | 2/- | 2/4r | 2/3r, without update, then with
//     780-1700   P = 8  0.98 | 1.00 | 0.99 | 1.04, 0.98 | 0.99 | 0.98 | 1.01
//                P = 12 0.96 | 0.98 | 0.96 | 1.01, 0.99 | 0.99 | 0.99 | 1.02
//                P = 24 0.99 | 1.00 | 0.95 | 0.99, 0.99 | 0.98 | 0.96 | 0.98
//                P = 64 1.00 | 1.01 | 0.94 | 0.96, 0.99 | 0.98 | 0.93 | 0.93
//     1900-7000  P = 8 - | - | 0.97 | 1.01, - | - | 0.97 | 0.98   P = 12 - | - | 0.95 | 0.99, - | - | 0.98 | 0.98
//     1000-2050 with update, 4/- | 4/3  P = 5 0.97 | 1.00   P = 6 0.98 | 0.98   P = 7 0.98 | 1.01
// Tensors shorter than a tile leave most parts empty: a workgroup takes whole tiles then.  900 elements each, P = 8  560 tiles fp32
// 13.3 -> 6.9 us, 2230 42 -> 20, bf16 2230 22 -> 21; P = 64  130 tiles 0.62.  A tile of several parts (long_tiles) keeps its workgroup
// up to four times as long, and a short launch with it: weights and short vectors, batch kernel = 1, whole tiles | four replicas and
// as many workgroups as fit, in parts, in rows, by the share of long tiles, means (worst) of P = 2 to 64, with and without update:
//   fp32  none 0.50 (0.85) | 0.90 (1.01)
//         2 to 7 %   below 700 tiles 1.07 (1.42) | 0.89 (1.12)   to 1600 0.82 (0.93) | 0.90 (0.96)   beyond 0.59 (0.65) | 0.89 (0.94)
//         7 to 15 %  below 700 tiles 1.23 (1.60) | 0.92 (1.29)   to 1600 0.88 (1.02) | 0.93 (0.99)   beyond 0.70 (0.75) | 0.94 (0.99)
//         15 to 30 % below 700 tiles 1.34 (1.70) | 0.94 (1.06)   beyond 1600 0.96 (1.22) | 0.94 (1.01)
//   bf16  none 0.92 (1.15) | 1.06 (1.44)
//         2 to 7 %   below 700 tiles 1.02 (1.22) | 0.86 (1.08)   to 1600 0.99 (1.17) | 1.00 (1.10)   beyond 0.98 (1.08) | 1.09 (1.16)
//   1 % (one to six of 505 tiles) fp32 P = 2 to 12 1.20 to 1.51 | 0.85 to 1.02;  3 % of 940 bf16 P = 24 with update 1.41 | 1.15
// Nor do few workgroups that share a CU, or two replicas, go with tiles that are less than half full: most have nothing to load and
// the others wait for room.  The rule for full tiles had up to 2.1 times the batch kernel's time there (P = 32 581 tiles 22.4 -> 31.4 us,
// 1500 tensors 1.4 and 2.0 at P = 16 to 64), this one 0.90 (4 replicas, 806 launches), the pass 0.97; below 320 tiles rows are not
// even (P = 64 219 tiles 1.29).  From 50 to 60 % full four replicas are still the better ones, 0.97 to 1.00 where 2/3r has 1.02 to
// 1.21, with rows where full tiles have them: elsewhere a pass is 1.05 with rows and 1.03 without (P = 2 to 8).
// Sixty-four items in a row on an XCD, 256 KiB of each replica, whose lines of the tile table its L2 then has, and whose pages its
// address translation: BERT-Large-shaped P = 8 bf16 5683 -> 6085 GB/s, with update 5787 -> 6063, BERT-Base-shaped P = 8 fp32 5731 ->
// 5909.
// Not where w of a launch fits the L2s (2048 tiles, 32 MiB): the all-gather behind it reads w in the L2 of the XCD that wrote it, if
// both go through the tiles as they fall.  Pass = reduce-scatter with update, all-gather, one state over and over / three in turn,
// batch kernel = 1, as they fall | in rows: fp32 P = 2 900 tiles 0.98 / 0.99 | 1.15 / 0.98, 1800 1.01 / 1.01 | 1.09 / 0.98, P = 8 600
// 1.03 / 1.02 | 1.07 / 1.02, 900 1.01 / 1.01 | 1.08 / 0.98, 1800 1.00 / 1.01 | 1.04 / 0.98, P = 16 400 1.02 / 1.02 | 1.04 / 1.02,
// 900 0.98 / 0.97 | 0.99 / 0.94; dear_iteration P = 8 800 1.02 / 1.03 | 1.13 / 1.03, bf16 P = 6 800 1.00 / 0.99 | 1.21 / 0.98; more
// replicas leave little of it: P = 32 fp32 900 0.98 / 0.96 | 0.95 / 0.92, 400 1.00 / 0.99 | 1.01 / 0.99.
// fp32 with 8 to 16 replicas, 6000 tiles and more: four replicas, two workgroups, as they fall, whose rows of several replicas do
// not drift apart.  Models' lists, 4/2 | 2/4r (without update) or 2/3r (with), and dear_iteration: ResNet-50-shaped (6342 tiles) P = 8
// 0.98 | 0.98, 1.00 | 0.99, 0.99 | 1.01, P = 12 0.97 | 0.98, 1.02 | 1.01, 0.99 | 0.99, P = 16 0.99 | 1.01, 0.99 | 0.98, 0.98 | 0.98;
// Inception-v4-shaped (10732) P = 8 0.99 | 0.97, 1.00 | 1.00, 0.97 | 0.99, P = 12 0.98 | 0.98, 1.01 | 1.00, 0.96 | 0.98, P = 16 0.99 |
// 1.00, 0.99 | 1.00, 0.95 | 0.96; BERT-Base-shaped (26988) P = 8 0.98 | 1.00, 0.99 | 0.99, 0.99 | 1.01, P = 16 0.99 | 1.03, 0.99 |
// 0.97, 1.00 | 0.99; below, DenseNet-201-shaped (5242) P = 8 0.97 | 0.92, 1.00 | 0.99, 0.99 | 0.97.  One tensor of 6000 to 13000 tiles
// likes rows (P = 8 with update 1.00 | 0.96).  bf16 from 6000 tiles on 2/3r: BERT-Large-shaped all buckets 2/4r 0.91, 2/3r 0.89, with
// update 0.95 and 0.94, 12000 to 40000 tiles P = 8 0.97 and 0.94, 1.00 and 0.98, P = 16 1.03 and 1.00, 1.01 and 0.99.
// In dear_iteration where the all-gather comes next (caches_w) four replicas a lane and as many workgroups as fit, below 1600 tiles
// (fp32 from 8 replicas on 2048): fp32 P = 8 350 / 550 / 800 / 1200 tiles 1.02 / 1.01 / 0.99 / 0.99, two replicas
// 1.03 / 1.02 / 1.00 / 0.99 and with four workgroups 1.07 / 1.04 / 1.02 / 1.00, P = 9 to 12 1600 two in rows 1.02 to 1.03; bf16 P = 6
// and 8 at 550 1.03 (the batch kernel up to 700), P = 9 to 20 320 to 450 1.02 to 1.05 (the rule without caches_w).  Beyond 2048 tiles
// 2/4r | 2/3r | 2/-r: 604 ragged tensors bf16 P = 5 0.99 | 1.01 | 1.01, P = 6 0.99 | 1.01 | 1.02, P = 7 0.97 | 0.98 | 0.99, P = 8 1.00
// | 1.00 | -, BERT-Large-shaped P = 8 0.98 | 0.98 | 0.99; fp32 ResNet-50-, Inception-v4- and DenseNet-201-shaped P = 4 0.99 | 0.98 |
// -, 1.00 | 1.00 | -, with gbar 1.03 | 1.01 | -, 0.99 | 1.01 | -, P = 5 1.00 | 1.00 | - and 1.00 | 1.01 | -, P = 7 1.01 | 1.02 | - and
// 0.99 | 1.01 | -.
inline reduce_scatter_shape reduce_scatter_shape_of(bool bf16, bool updates, bool caches_w, int64_t P, int64_t elems, int64_t tiles,
                                                    int64_t long_tiles, int64_t cut_tiles)
{
    auto depth = [&](int most) { return P >= most ? most : P >= 4 ? 4 : P >= 2 ? 2 : 1; };
    auto filled = [&](int percent) { return elems * 100 >= tiles * DEAR_TILE_ELEMS * percent; };
    const int run = tiles < (P <= 8 ? 2048 : P <= 16 ? 1600 : 320) ? 0 : 6;
    auto parts = [&](int most, int residency) { return reduce_scatter_shape{depth(most), residency, run, false}; };
    const reduce_scatter_shape batch{0, 0, 0, false};
    const bool full = filled(85), cut = cut_tiles * 8 >= tiles;
    if (tiles >= (P >= 8 ? 96 : 128) && !filled(50) && long_tiles * (bf16 ? 15 : 7) <= (tiles < 1600 ? 0 : tiles))
        return {depth(8), 0, 4, true};
    if (!bf16 && full && P >= 8 && P <= 16 && tiles >= 6000) return {4, 2, 0, false};
    if (caches_w && P >= 4 && filled(50)) {
        if (bf16 && P <= 8 && tiles < 700 && tiles >= (P % 4 ? 40 : 110)) return batch;
        if (tiles >= 256 && tiles < (bf16 || P < 8 ? 1600 : 2048) && P <= (bf16 ? 8 : 16)) return {4, 0, 0, false};
        if (tiles >= (bf16 ? 1600 : 2048)) return parts(2, tiles < 2048 ? 0 : !bf16 && P == 4 ? 3 : 4);
    }
    if (!(caches_w && tiles >= 256 && (bf16 ? P >= 4 && P <= 8 : true)) && batch_kernel_stays(bf16, updates, P, tiles, cut)) return batch;
    if (tiles >= 128 && !filled(60)) return {depth(4), 0, filled(50) ? run : tiles < 320 ? 0 : 6, false};
    if (P < 4) return parts(2, updates && (full || bf16) && tiles >= (bf16 ? 512 : P > 1 ? 4096 : 1024) ? 4 : 0);
    if (!bf16 && P > 4 && P <= 16 && tiles >= 320 && tiles < (P < 12 ? 1024 : 700)) return {4, 0, 0, false};
    if (bf16 && P <= 16 && (P >= 8 || !updates) && tiles >= (P < 8 ? 900 : 750) && tiles < (P <= 8 ? 2048 : 1600)) return {4, 0, 0, false};
    if (P < 8) {
        if (bf16 && updates) return parts(4, tiles >= 2048 || (tiles >= 1024 && cut_tiles * 16 >= tiles) ? 3 : 0);
        if (P == 4 ? !bf16 && tiles < 75 : tiles < (bf16 ? 256 : 160)) return parts(4, 0);
        if (updates) return parts(2, full && tiles >= 2048 ? 3 : 0);
        return parts(2, full && tiles >= 4096 ? 4 : 0);
    }
    if (tiles < (!bf16 ? 64 : P < 24 ? 110 : 132)) return parts(8, 0);
    if (tiles < (bf16 ? 288 : 128)) return parts(4, 0);
    if (tiles < (bf16 ? 750 : P > 16 ? 400 : 512)) return parts(2, 0);
    if (bf16) return parts(2, tiles >= 6000 ? 3 : 4);
    if (!full && P < 13 && tiles < 2048) return parts(2, 0);
    return parts(2, (P >= 24 ? tiles >= 512 : updates && (P >= 13 || tiles >= 2048)) ? 3 : 4);
}

// Whether a replica's workgroups take two parts in a row (1) or each the next one (0) on an XCD (see all_gather_kernel): two are
// what a workgroup of a bf16 reduce-scatter + update in halves of tiles wrote, and where that launch comes right before, as in
// dear_iteration, they are in this XCD's L2.  The more replicas, and the emptier the tiles, the more the rounding to 16 parts costs.
// One / two in a row:
//   dear_iteration, us, one bucket of 100 / 200 / 400 / 850 full tiles  P = 8 8.5 / 8.3  12.6 / 12.1  22.1 / 20.1  39.5 / 38.4
//     P = 24 16.0 / 16.0  24.7 / 24.2  45.9 / 44.4  92.3 / 88.7   P = 40 23.4 / 24.4  36.8 / 37.2  71.6 / 69.5  144 / 145
//     P = 48 28.5 / 28.9  43.9 / 45.2  82.5 / 83.1   P = 64 38.7 / 39.4  57.4 / 59.0  108 / 109  225 / 221
//   the same, weights and short vectors, change in %: P = 3 -7 to 0, P = 8 up to 150 tiles 0, 340 to 430 full ones -4 to -8,
//     P = 12 and 16 up to 230 tiles +1 to +3, 390 full ones -4, P = 24 +1 to +3, P = 32 +1 to +4, P = 48 and 64 +3 to +5
//   all reduce-scatters, then all all-gathers, change of the whole pass in %, eight buckets or fewer of 40 / 100 / 200 / 400 / 850
//   full tiles
//     P = 4 -7 / -3 / -2 / 0 / 0   P = 8 -9 / -4 / 0 / 0 / -1   P = 16 -3 / -2 / 0 / +1 / -2   P = 24 0 / 0 / +2 / +2 / -1
//     P = 32 +1 / +1 / +2 / +3 / -1   P = 48 -1 / +1 / +3 / +3 / -1   P = 64 +2 / +3 / +3 / +3 / +3
//   the same, weights and short vectors: P = 3 and 4 -6 to 0, P = 8 -3 to +2, with an update between +1 to +2.5,
//     P = 12 and 16 +1 to +3, from P = 24 on +2 to +5
// Beyond 1024 tiles where the launch before goes in halves of tiles as they fall; one / two in a row, dear_iteration, cold, change of
// the whole pass against the batch kernel's in %, 1140 ragged tiles, 1200 of one tensor, 1520 ragged: P = 4 -5 / -8, -2 / -8, -5 / -9,
// P = 6 -3 / -8, 0 / -2, -2 / -5, P = 8 -2 / -4, 0 / 0, -2 / -4, P = 12 -2 / -4, -1 / 0, -3 / -4, P = 16 -1 / -2, +1 / +3, 0 / -2;
// calls of their own 0 / +1.
// Up to 1024 tiles also where that launch goes in rows (P = 24 660 full tiles +3 / 0, 910 +3 / 0, ragged 630 -2 / -1, 880 0 / -1,
// weights and short vectors 660 -1 / 0, P = 32 670 and 930 full +5 / 0).
inline unsigned all_gather_run(int grad_bytes, bool caches_w, int64_t max_workgroups, int64_t P, int64_t elems, int64_t tiles,
                               int64_t whole, int64_t long_tiles, int64_t cut_tiles, int64_t n_workers, bool behind_update)
{
    if (grad_bytes != 2 || max_workgroups > 0 || tiles >= 2048 || !half_tiles_filled(elems, tiles, whole)) return 0;
    if (!behind_update) return n_workers <= (tiles <= 160 ? 8 : tiles <= 1024 ? 4 : 0);
    if (tiles > 1024) {
        const reduce_scatter_shape s = reduce_scatter_shape_of(true, true, caches_w, P, elems, tiles, long_tiles, cut_tiles);
        return s.depth > 0 && s.run == 0 && !s.tiles && n_workers <= 12;
    }
    return n_workers <= 8 || (elems * 4 >= tiles * (3 * DEAR_TILE_ELEMS) && n_workers <= (tiles < 400 ? 32 : 47));
}

// Whether the entries of a pointer table lie within 32 bits of its beginning, as reduce_scatter_kernel counts them.
inline bool pointer_table_fits(int64_t P, int64_t L) { return P * L < int64_t{1} << 29; }

// dear_iteration handles consecutive buckets together until they hold this many tiles (32 Mi elements, 128 MiB of w).
// A launch costs about 2 us of ramp and drain, which shows up to some hundred microseconds; a longer group has more
// w for the last-level cache and a longer way back to it.  us per iteration with gbar, one launch pair per bucket / 2048 /
// 4096 / 8192 / 16384 / 32768 tiles (spread 0.1-1.4 %): ResNet-50-shaped P = 8 386 / 386 / 365 / 354 / 353 / 353, 58 tensors in
// 0.3 MB buckets P = 24 1198 / 955 / 969 / 964 / 964 / 961, BERT-Base-shaped in 16 MB P = 8 1867 / 1630 / 1575 / 1579 / 1566
// / 1578, P = 64 10016 / 10254 / 9642 / 9599 / 9532 / 9726, in 25 MB P = 16 2798 / 2799 / 2773 / 2760 / 2789 / 2825,
// BERT-Large-shaped bf16 in 25 MB P = 2 2077 / 2076 / 2070 / 2033 / 2044 / 2068, in 64 MB (a bucket each up to 8192) P = 8
// 3810 / 3852 / 3860.
constexpr int64_t ITERATION_TILES = 8192;

// Whether a group's reduce-scatter stores w with the ordinary cache policy, for the all-gather behind it: where w is
// still in the 256 MB last-level cache by then.  That takes a w which fits (a larger bucket is a group of its own),
// and little gradient traffic beside it, grad_bytes * P per element, or a w of all buckets that stays in the cache.
// us per iteration without gbar, non-temporal w / ordinary w (spread 0.1-0.3 %), P:
//   several groups, fp32  2 659 / 665   4 926 / 916  6 1175 / 1187  8 1447 / 1483  16 2593 / 2677  64 9483 / 9666
//                         (BERT-Base-shaped, 64 MB buckets);  Inception-v4-shaped 8 595 / 619
//   several groups, bf16  2 1807 / 1772  4 2460 / 2393  8 3671 / 3601  12 4910 / 4877  16 6109 / 6184
//                         (BERT-Large-shaped, 64 MB);  BERT-Base-shaped 24 2849 / 2919
//   one group, fp32       DenseNet-201-shaped 8 274 / 267, 16 488 / 487;  ResNet-50-shaped 8 346 / 347, 32 1173 / 1181
//   one group, bf16       ResNet-50-shaped 16 493 / 488, 32 941 / 921;  604 ragged tensors 7 203 / 190
//   one bucket beyond ITERATION_TILES, 110 M  fp32 2 686 / 683  8 1492 / 1529  64 9396 / 9706; bf16 8 1213 / 1215
inline bool iteration_caches_w(int grad_bytes, int64_t P, int64_t group_tiles, int64_t all_tiles)
{
    constexpr int64_t ALL_CACHED_TILES = 7168;  // 112 MiB of w
    if (group_tiles > ITERATION_TILES) return false;
    if (grad_bytes * P <= (grad_bytes == 2 ? 24 : 16)) return true;
    return grad_bytes * P <= 64 && all_tiles <= ALL_CACHED_TILES;
}

// A bucket beyond ITERATION_TILES is handled in pieces of its tiles, whatever layers and shards they belong to, if that
// leaves each piece's w in the last-level cache for its all-gather.  us per iteration without and with gbar, one launch pair /
// pieces, one bucket (two runs of one side differ by up to 5 %): bf16 P = 3 50 M 321 / 295 and 370 / 338, 100 M 640 / 586 and
// 740 / 674, P = 4 50 M 369 / 344 and 419 / 386, P = 5 36 M 295 / 281 and 332 / 312, P = 6 60 M 543 / 511 and 610 / 561, P = 8 50 M
// 536 / 524 and 577 / 554, 110 M 1155 / 1128 and 1263 / 1197; with a bounded grid of 256 P = 3 50 M 336 / 322 and 385 / 365, P = 8 110
// M 1442 / 1328 and 1537 / 1404, of 1024 P = 8 60 M 803 / 724.
// Not where w is stored non-temporally anyway: bf16 P = 16 100 M 1766 / 1768 and 1868 / 1848, fp32 P = 5 36 M 336 / 344 and 359 / 366,
// P = 8 100 M 1284 / 1312 and 1370 / 1388.  Pieces of 4096 and 12288 tiles are level to 1 %.
inline int64_t iteration_pieces(int grad_bytes, int64_t P, int64_t group_tiles, int64_t all_tiles)
{
    if (!iteration_caches_w(grad_bytes, P, ITERATION_TILES, all_tiles) || grad_bytes != 2) return 1;
    return (group_tiles + ITERATION_TILES - 1) / ITERATION_TILES;
}

// Whether a group whose gbar is wanted takes three launches, the update behind the reduce-scatter: the more replicas
// are read, the less it costs to read gbar once more, and the better the reduce-scatter runs with one output instead
// of three.  us per iteration, one kernel / two (spread 0.2-2 %), fp32 P: BERT-Base-shaped, 64 MB buckets 8 1549 / 1638,
// 16 2715 / 2695, 24 3888 / 3820, 32 5097 / 4980, 64 9649 / 9504; one bucket of 110 M 64 9807 / 9517; ResNet-50-shaped
// 16 644 / 644, 32 1209 / 1184, 64 2340 / 2277; 2 M elements 24 73.4 / 75.7, 64 192 / 192; bf16: BERT-Base-shaped
// 24 2949 / 2955, 32 3841 / 3817, 64 7542 / 7346; 8 M elements 64 555 / 545.
inline bool iteration_updates_apart(int grad_bytes, int64_t P, int64_t group_tiles)
{
    return grad_bytes * P >= 96 && group_tiles >= 2048;
}

// Whether dear_iteration takes everything in ONE launch, each workgroup storing the new w of its elements to all replicas.
// That saves a launch (2 us of GPU time, 3 of the host's), the 4-byte re-read of w, and the all-gather's empty workgroups
// for the parts of tiles that short tensors leave open (`open` elements); but the replicas are written as P interleaved
// streams.  As long as the writes go to the 256 MB last-level cache that does not matter; HBM takes it the worse the more
// streams there are, and from large calls with few replicas the re-read costs more.  GPU time, us, without gbar, two launches / one
// (three sets of buffers in turn, spread 1 %):
//   fp32  P = 2 0.2 M elements 5.7 / 4.1  1 M 8.9 / 6.9  4 M 25.7 / 22.9  10 M 55.6 / 53.2  40 M 237 / 207  100 M 607 / 512
//         P = 3 1 M 10.0 / 8.3  4 M 30.0 / 28.6  6 M 41.2 / 41.7  20 M 129 / 129  30 M 208 / 194  100 M 720 / 639
//         P = 4 1 M 11.3 / 9.8  3 M 26.8 / 26.8  6 M 48.1 / 50.0  20 M 155 / 160  50 M 402 / 383 (with gbar 429 / 430)
//         P = 8 0.2 M 7.5 / 6.7  1 M 15.9 / 15.2  1.5 M 22.2 / 22.8  6 M 78.8 / 85.5  P = 12 0.5 M 13.4 / 13.2  1 M 22.6 / 23.8
//         P = 16 0.2 M 11.3 / 11.8  1 M 27.1 / 30.8
//         P = 8 from 6 to 9 M copied elements, where only 240 to 258 tiles, of four workgroups each, fill the 256 CUs evenly: one
//         tensor 223 tiles 13.1 / 14.1  242 13.7 / 13.3  258 14.9 / 13.8  262 15.8 / 16.1  277 16.0 / 17.2, 23 tensors 230 14.3 / 14.2
//         248 15.4 / 14.3  257 15.6 / 14.4  267 16.5 / 16.7  281 16.9 / 17.4
//         open tiles: P = 8 1 M in 500 tensors 27.3 / 22.4, 2 M in 200 34.2 / 34.1, 3 M in 500 50.2 / 50.7
//                     P = 16 1 M in 500 47.8 / 39.7, in 60 29.0 / 32.0, 3 M in 500 86.3 / 93.2
//   bf16  P = 2 1 M 8.9 / 6.6  6 M 33.4 / 31.0  20 M 92.2 / 97.1  30 M 150 / 145  100 M 514 / 481
//         P = 4 1 M 10.7 / 8.7  3 M 24.1 / 22.8  6 M 42.8 / 43.9  P = 8 0.5 M 10.3 / 9.2  1.5 M 19.3 / 18.5  3 M 34.3 / 35.2
//         P = 12 0.5 M 13.2 / 12.8  1 M 18.6 / 19.2  P = 16 0.2 M 11.2 / 11.9  1 M 22.9 / 25.3, in 500 tensors 46.2 / 37.7
// From 9 (bf16) or 10 replicas on a launch of few tiles is slower so: each of its few workgroups writes them all, one after another.
// One launch behind start of the two, GPU time without gbar:
//   fp32  P = 12 20 tiles 7.5 / 8.1  33 6.8 / 6.2   P = 16 26 tiles 7.7 / 8.6  46 9.0 / 9.3  61 9.8 / 9.6
//         P = 32 42 tiles 12.2 / 15.3  77 17.3 / 17.8  92 18.4 / 17.8   P = 64 72 tiles 25.1 / 27.8  94 32.9 / 32.4
//   bf16  P = 8 18 tiles 5.0 / 5.2  39 5.4 / 5.2   P = 10 18 tiles 5.5 / 6.1  40 8.6 / 8.7  76 9.9 / 9.5
//         P = 16 46 tiles 9.4 / 10.0  76 10.8 / 10.5
//         P = 32 62 tiles 15.6 / 17.2  92 18.5 / 18.3  112 20.6 / 18.9   P = 64 94 tiles 32.3 / 31.9  124 37.5 / 33.1
// And bf16 beyond what the last-level cache holds of the pass's elems * (6 P + 20) bytes: tensors of 2000 elements P = 8 2 M
// without / with gbar 44 / 38 and 48 / 45, 6 M 99.8 / 100 and 112 / 125, P = 32 0.6 M 44 / 40, 2 M 108 / 130, P = 64 0.3 M in 18
// 47.5 / 49.3, 2 M 212 / 254; of 2600 P = 6 2.6 M 39.9 / 40.7 and 44.7 / 48.5, P = 8 0.8 M 17.0 / 15.4, 2.6 M 46 / 50 and 51 / 58;
// whole P = 5 2 M (493 tiles) 17.2 / 15.8, 2.1 M (517) 18.2 / 19.7, P = 4 2.3 M (566) 17.6 / 18.9, 3 M (737) 23.1 / 21.0; weights and
// short vectors P = 5 4 M (71 %) 41.8 / 39.2, P = 8 1.7 M (88 %) 22.5 / 21.4, P = 11 1.3 M (51 %) 34.4 / 31.0 and 35.9 / 33.4.  Of
// 1500 and less one launch is faster at any size (P = 8 4.5 M 90 / 65, P = 32 1.5 M 102 / 94), as in fp32 (P = 64 1.5 M 272 / 266),
// where half full tiles cost from 25 replicas on (135 tensors of 3500 in 246 tiles P = 64 75.7 / 78.7, 1 M in 500 160 / 169; weights
// and short vectors 40 % full P = 64 52.5 / 59.3).
inline bool iteration_gathers_at_once(int grad_bytes, int64_t P, int64_t elems, int64_t tiles, bool with_gbar, int64_t max_workgroups)
{
    constexpr int64_t M = 1000000;
    if (max_workgroups > 0 || tiles * AG_SPLIT > MAX_GRID) return false;
    const bool bf16 = grad_bytes == 2;
    const int64_t few = bf16 ? (P < 31 ? 4 * P : 124) : P <= 12 ? 2 * P : P < 31 ? 3 * P : 92;
    if (P > (bf16 ? 8 : 9) && tiles < few) return false;
    const int64_t open = tiles * DEAR_TILE_ELEMS - elems;
    const bool even = P == 8 && tiles >= 240 && tiles <= 258;
    const int64_t cached = P > 12 ? 0 : bf16 ? (P > 8 ? 7 : 12) * M : (P < 8 || even ? 9 : 6) * M;
    if (P * (elems - open) <= cached) {
        if (elems * 5 < tiles * (2 * DEAR_TILE_ELEMS)) return true;
        if (!bf16) return P <= 24 || elems * 8 < tiles * (3 * DEAR_TILE_ELEMS);
        if (P >= 3 && tiles > 512 && tiles <= 680 && elems * 4 >= tiles * (3 * DEAR_TILE_ELEMS)) return false;  // a third whole tile for few of the CUs
        const int64_t most = elems * 5 >= tiles * (3 * DEAR_TILE_ELEMS) ? 120 : elems > open ? 180 : 256;
        return P < 6 || (P <= 32 && elems * (6 * P + 20) <= most * M);
    }
    if (bf16) return P <= 2 && elems >= 25 * M;
    return P <= 2 || (P == 3 && elems >= 25 * M) || (P == 4 && elems >= (with_gbar ? 64 : 40) * M);
}

// Workgroups that may share a CU in such a launch, 0 for as many as fit: HBM serves many streams at once better the fewer loads
// compete, in launches long enough for it and whose tiles are four fifths full.  us at as many / 2 / 1, fp32
// with gbar P = 2 5 M 32.8 / 31.6 / 38.9, 100 M 640 / 579 / 703, P = 3 100 M 788 / 722 / 878, without P = 4 100 M 854 / 776 / 876;
// bf16 with gbar, half tiles, P = 2 30 M - / 180 / 161, 100 M 596 / 594 / 525.  bf16 P = 1 without gbar 26 M 97 / 93 / 106, 100 M
// 389 / 355 / 395, 250 M - / 923 / 1017, with it 26 M 125 / 114 / 118, 80 M - / 354 / 358, 100 M 499 / 449 / 444, 150 M - / 702 / 683.
inline int iteration_at_once_residency(bool bf16, bool with_gbar, int64_t P, int64_t elems, int64_t tiles)
{
    if (elems * 5 < tiles * (4 * DEAR_TILE_ELEMS)) return 0;
    if (bf16) return elems < 25000000 ? 0 : P == 1 && !(with_gbar && elems >= 90000000) ? 2 : 1;
    return elems >= 4000000 ? 2 : 0;
}

// bf16, half tiles a workgroup in such a launch: where whole ones would leave the 256 CUs unevenly filled (P = 4 0.5 M
// 7.2 / 6.3, 1.5 M 13.4 / 12.3, 2 M 15.0 / 15.7, P = 8 0.5 M 10.1 / 9.2, 1.5 M 19.9 / 18.5, 2 M 24.3 / 24.7), and in large ones (P = 2
// 100 M 599 / 525 with one workgroup per CU or as many as fit, which is what each likes best).
inline bool iteration_at_once_half_tiles(int64_t elems, int64_t tiles)
{
    return tiles <= 400 || elems >= 25000000;
}
