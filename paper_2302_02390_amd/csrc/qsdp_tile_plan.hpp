// Launch shape of the tile kernels (qsdp_tile_kernel.hpp) for a bucket size. Plain C++, no HIP: the host side uses
// it to launch, and it can be compiled and checked without a GPU.
#pragma once

#include <stdint.h>

namespace qsdp {

// A team of `waves` waves holds `rows` rows of 64 * waves slots of four elements, i.e. 8 * waves * rows groups of
// eight slots (32 elements). A bucket of 32 * k elements is k consecutive groups; a tile is as many whole buckets
// as fit.
struct TilePlan {
    int waves, rows;
    int buckets;           // whole buckets per tile
    int lanes_log2;        // lanes that combine one bucket's group minima and maxima: 2^lanes_log2
    uint32_t group_magic;  // bucket of group i of the tile = (i * group_magic) >> 16
};

constexpr int kTileMaxRows = 8;

inline int tile_groups(int waves, int rows) { return 8 * waves * rows; }

inline TilePlan tile_plan_for(int bucket, int waves, int rows) {
    TilePlan t = {};
    const int k = bucket / 32;
    t.waves = waves;
    t.rows = rows;
    t.buckets = tile_groups(waves, rows) / k;
    // as many lanes per bucket as the team has for each, at most a wave and at most one per group
    while ((2 << t.lanes_log2) <= 64 && (2 << t.lanes_log2) <= 64 * waves / (t.buckets > 0 ? t.buckets : 1) &&
           (1 << t.lanes_log2) < k)
        ++t.lanes_log2;
    // i < 256 and k <= 256: i * (65536 / k + e), e < 1, is off by less than 65536 / k from a multiple
    t.group_magic = (65536u + (uint32_t)k - 1u) / (uint32_t)k;
    return t;
}

// Which shape a bucket size gets. A tile that whole buckets do not fill computes on idle slots, so the fuller one
// wins; a tile of one wave needs no barriers and fewer registers, so a larger one has to be fuller by a tenth.
inline TilePlan tile_plan(int bucket) {
    static const int shapes[6][2] = {{1, 4}, {1, 6}, {1, 8}, {4, 4}, {4, 6}, {4, 8}};
    TilePlan best = {};
    double best_fill = 0.0;
    for (const auto& s : shapes) {
        const TilePlan t = tile_plan_for(bucket, s[0], s[1]);
        const double fill = (double)t.buckets * (bucket / 32) / tile_groups(s[0], s[1]);
        if (fill > 1.1 * best_fill) {
            best = t;
            best_fill = fill;
        }
    }
    return best;
}

// ceil(2^18 / bits): slot of the first bit of word w of a tile's code stream = (8 * w * magic) >> 18. A tile has at
// most 2^11 slots, so 8 * w < 2^11 * bits and the product stays below 2^30.
inline uint32_t word_magic(int bits) { return (262144u + (uint32_t)bits - 1u) / (uint32_t)bits; }

}  // namespace qsdp
