// Host-only check (dear_internal.h, plan.cpp): where each XCD takes an eighth of a chunk, every part belongs to exactly one workgroup, in
// whole chunks and in last ones; the rule takes no short launch and none of mostly empty tiles; and replicas are found alike where
// seven eighths of the elements lie alike on lines.  Exits non-zero on the first mistake.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "dear_internal.h"

// What dear_mark_runs says of three replicas whose tensors begin so many elements behind a line: starts[p][layer].
static bool alike(const std::vector<int64_t> &sizes, const std::vector<std::vector<int>> &starts)
{
    dear_plan_t *plan = nullptr;
    const int32_t L = static_cast<int32_t>(sizes.size()), P = static_cast<int32_t>(starts.size());
    if (dear_plan(sizes.data(), L, P, DEAR_NO_LIMIT, 4, &plan) != DEAR_OK) std::exit(1);
    std::vector<float *> params;  // addresses only
    for (int32_t p = 0; p < P; ++p)
        for (int32_t l = 0; l < L; ++l)
            params.push_back(reinterpret_cast<float *>((uintptr_t(p + 1) << 40) + (uintptr_t(l) << 32) + 4 * uintptr_t(starts[p][l])));
    int64_t n_tiles = 0;
    const int64_t n_runs = dear_emit_runs(*plan, 0, plan->B, nullptr, 0, &n_tiles, nullptr);
    std::vector<dear_run> runs(n_runs);
    dear_emit_runs(*plan, 0, plan->B, runs.data(), n_runs, &n_tiles, nullptr);
    const bool said = dear_mark_runs(*plan, params.data(), runs.data(), n_runs);
    dear_plan_free(plan);
    return said;
}

static bool replicas()
{
    const int64_t M = 960000;  // three shards of 78 tiles and more
    const std::vector<int64_t> one{M};
    if (!alike(one, {{0}, {0}, {0}}) || !alike(one, {{4}, {4}, {4}}) || !alike(one, {{28}, {28}, {28}})) return false;
    if (alike(one, {{0}, {12}, {20}}) || alike(one, {{4}, {4}, {0}})) return false;
    // an eighth of the elements lies differently, and a little more of them
    if (!alike({M / 8, M / 8 * 7}, {{0, 0}, {4, 0}, {8, 0}}) || alike({M / 8 + 8, M / 8 * 7 - 8}, {{0, 0}, {4, 0}, {8, 0}})) return false;
    // short runs are not moved: alike only where they begin on lines
    const std::vector<int64_t> many(60, 16000);
    auto all = [&](int start) { return std::vector<std::vector<int>>(3, std::vector<int>(many.size(), start)); };
    return alike(many, all(0)) && !alike(many, all(4));
}

int main()
{
    if (!replicas()) {
        std::fprintf(stderr, "FAILED replicas alike\n");
        return 1;
    }
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
        for (int64_t tiles : {1, 900, 959, 960, 1599, 1600, 2047, 2048, 4999, 5000, 5999, 6000, 30000}) {
            const bool long_enough = tiles >= (P >= 24 ? 960 : P >= 12 ? 1600 : 2048) && P >= 3 && (P >= 5 || tiles < 5000);
            const int64_t room = tiles * DEAR_TILE_ELEMS, least = tiles < 6000 ? room / 8 * 7 : room / 2;
            if (all_gather_in_eighths(room, tiles, P) != long_enough || all_gather_in_eighths(least, tiles, P) != long_enough ||
                all_gather_in_eighths(least - 1, tiles, P)) {
                std::fprintf(stderr, "FAILED rule tiles=%lld P=%lld\n", (long long)tiles, (long long)P);
                return 1;
            }
        }
    std::printf("all_gather_eighths: ok\n");
    return 0;
}
