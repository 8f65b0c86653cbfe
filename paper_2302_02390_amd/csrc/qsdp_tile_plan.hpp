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

// Lets a tile take only `buckets` buckets (at least one of them).
inline void tile_take(TilePlan& t, int bucket, int buckets) {
    t.buckets = buckets;
    // as many lanes per bucket as the team has for each, at most a wave and at most one per group
    t.lanes_log2 = 0;
    while ((2 << t.lanes_log2) <= 64 && (2 << t.lanes_log2) <= 64 * t.waves / (buckets > 0 ? buckets : 1) &&
           (1 << t.lanes_log2) < bucket / 32)
        ++t.lanes_log2;
}

inline TilePlan tile_plan_for(int bucket, int waves, int rows) {
    TilePlan t = {};
    const int k = bucket / 32;
    t.waves = waves;
    t.rows = rows;
    tile_take(t, bucket, tile_groups(waves, rows) / k);
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

// ... for a call that leaves most of the chip idle: the smallest team that holds a bucket, and no more buckets than
// fill its first row if that holds one (the arithmetic of an unused second row is left out). What bounds such a call
// is the instructions of a single wave.
inline TilePlan tile_plan_small(int bucket) {
    static const int shapes[5][2] = {{1, 2}, {4, 2}, {4, 4}, {4, 6}, {4, 8}};
    const int k = bucket / 32;
    int i = 0;
    while (tile_groups(shapes[i][0], shapes[i][1]) < k) ++i;
    TilePlan t = tile_plan_for(bucket, shapes[i][0], shapes[i][1]);
    const int row = tile_groups(t.waves, 1);
    if (k <= row) tile_take(t, bucket, row / k);
    return t;
}

// ... for tensors of `mean` buckets with a level table each, where a tile of many buckets would give one team table
// after table: the smallest team that holds a bucket, of one wave if that can be, and no more buckets than a tensor
// has.
inline TilePlan tile_plan_tensors(int bucket, uint64_t mean) {
    static const int shapes[7][2] = {{1, 2}, {1, 4}, {1, 6}, {1, 8}, {4, 4}, {4, 6}, {4, 8}};
    int i = 0;
    while (tile_groups(shapes[i][0], shapes[i][1]) < bucket / 32) ++i;
    TilePlan t = tile_plan_for(bucket, shapes[i][0], shapes[i][1]);
    if (mean < (uint64_t)t.buckets) tile_take(t, bucket, mean > 0 ? (int)mean : 1);
    return t;
}

// The tile of a call of `num_buckets` buckets. Fewer than four waves to each of the chip's 1024 SIMDs leave it idle.
// Measured (us, buckets of 224 and 608, the fuller tile against the small one): 2^18 elements AdamW step 19.4 / 7.6
// and 16.4 / 7.9, encoder 7.2 / 3.9 and 6.7 / 4.1, receive side from 8 peers 24 / 10 and 21 / 11; 2^20 elements in
// buckets of 416 1.04-1.3 times faster, in buckets of 32 and 96, which are past the line, 0.9-1.1 times.
// tensors: how many level tables the call has (0: not one per tensor). most_waves: of a launch.
inline TilePlan choose_tile(int bucket, uint64_t num_buckets, uint64_t tensors, uint64_t most_waves) {
    const TilePlan full = tile_plan(bucket);
    if (tensors > 0 && num_buckets / tensors < (uint64_t)full.buckets)
        return tile_plan_tensors(bucket, num_buckets / tensors);
    const TilePlan small = tile_plan_small(bucket);
    const uint64_t tiles = (num_buckets + (uint64_t)small.buckets - 1) / (uint64_t)small.buckets;
    const uint64_t waves = tiles * (uint64_t)small.waves;
    return waves < 4096 && waves < most_waves ? small : full;
}

// What a mode is bound by in a full tile.
enum TileWork {
    TILE_MEMORY,        // the weight encoder, the steps; the code-resident one and the receive side are bound by both
    TILE_INSTRUCTIONS,  // the gradient encoder
    TILE_ADAMW,         // long chains of divisions: more waves in flight for longer
};

// ... for a call of middling size: two rows of a team of four, all buckets that fit (buckets of at most 2048).
inline TilePlan tile_plan_half(int bucket) { return tile_plan_for(bucket, 4, 2); }

// The tile of a call without learned levels. Between the two plans above lies a range in which the small tile would be
// too many half-empty waves and the full one too few waves: from one to six waves of the half tile to a SIMD, or
// twelve with AdamW. Measured (us, the plan of choose_tile / half; buckets of 96, 416, 544, 1504): step, 2^19 elements
// 7.2 / 6.6, 6.9 / 6.6, 8.2 / 6.9, 7.5 / 7.2, 2^20 9.1 / 7.5, 8.1 / 7.7, 9.6 / 8.4, 8.3 / 8.2, 2^21 10.5 / 9.6, 10.6 /
// 9.3, 11.4 / 10.5, 12.1 / 10.8, 2^22 13.4 / 14.3, 13.6 / 15.1, 14.1 / 16.1, 14.3 / 16.2; AdamW step, 2^20 15.8 / 11.8,
// 12.5 / 11.8, 16.9 / 12.9, 13.1 / 12.9, 2^22 27.3 / 25.7, 27.3 / 26.6, 28.1 / 27.6, 28.0 / 28.2. Below, at 2^16, the
// small tile is 0-6 % faster (eight peers with AdamW 9.2 against 11.1).
// The gradient encoder, which instructions bind, shares what a tile costs among six rows rather than four where these
// are as full (2^25 elements, buckets of 96, 416, 544 31.8 / 28.7, 31.6 / 29.8, 31.6 / 29.5), from four waves of
// theirs to a SIMD on (2^22, bucket 160, from 16 bits 8.7 / 9.2). Others do not gain: steps bound by memory 74.0 /
// 75.1, 74.3 / 75.4, 76.1 / 75.5, the code-resident step 3-5 % where codes are of 8 bits, losing up to 8 % at 5 bits,
// the receive side at no size (two peers, 2^22.6 elements in buckets of 32, 160, 544 15.9 / 18.4, 16.1 / 18.9, 17.3 /
// 18.4, eight peers, 2^25, 96, 544 105 / 108, 105 / 108).
// Over tensors the tile of choose_tile stays, unless the other one holds fewer buckets or the tensors are very large:
// a tile that meets a tensor's end is not contiguous and goes element by element, all of it, so small tensors make a
// larger tile slower throughout, and large ones end such a call late (us, the plan of choose_tile / the larger tile:
// 2^19 elements in tensors of one bucket of 32 / forty of 96, steps 9.1 / 13.4, 6.3 / 8.8, AdamW steps 12.0 / 16.5,
// 8.3 / 13.2; 2^23 in tensors of one bucket of 32, gradient encoder 35.0 / 49.2). Two rows with 4 buckets of 416 in
// place of four with 9 are 1.1-1.8 times faster at 2^21 elements, in tensors of 1 to 500 buckets. Six rows of the
// gradient encoder, 4 bits in buckets of 160, tensors of 128 and 512 tiles that end in a short bucket: 2^23 elements
// 13.5 / 15.8, 10.8 / 11.5, 2^25 38.1 / 38.2, 35.2 / 33.5, 100 * 2^20 101 / 101, 96 / 85.
inline TilePlan choose_step_tile(int bucket, uint64_t num_buckets, uint64_t most_waves, TileWork work,
                                 uint64_t tensors) {
    const TilePlan t = choose_tile(bucket, num_buckets, 0, most_waves), full = tile_plan(bucket);
    if (bucket <= 32 * tile_groups(4, 2)) {
        const TilePlan half = tile_plan_half(bucket);
        const uint64_t waves = (num_buckets + (uint64_t)half.buckets - 1) / (uint64_t)half.buckets * 4;
        if (waves >= 1024 && waves < (work == TILE_ADAMW ? 12288u : 6144u) && waves < most_waves &&
            (tensors == 0 || half.buckets < t.buckets))
            return half;
    }
    if (work == TILE_INSTRUCTIONS && t.rows == full.rows && t.waves == full.waves && t.buckets == full.buckets &&
        t.rows == 4) {
        const TilePlan six = tile_plan_for(bucket, 4, 6);
        const uint64_t waves = (num_buckets + (uint64_t)six.buckets - 1) / (uint64_t)six.buckets * 4;
        // as full: buckets a row, six rows against four
        const bool as_full = 100 * six.buckets * tile_groups(full.waves, 4) >= 95 * full.buckets * tile_groups(4, 6);
        const bool few_ends = waves >= 20480 && num_buckets >= 512 * tensors * (uint64_t)six.buckets;
        if (as_full && (tensors == 0 ? waves >= 4096 : few_ends)) return six;
    }
    return t;
}

// Whether a step on a flat vector, two fp32 operands in, weights and 8-bit codes on their min-max grids out, streams
// faster with three workgroups to a compute unit than with the four that the registers of six rows allow: large vectors
// in full tiles. us, four / three, buckets of 384, 768, 3040, where the tile is full: 96 * 2^20 elements 221 / 220, 220
// / 218, 220 / 217, 125M 275 / 270, 278 / 266, 273 / 267, 300 * 2^20 710 / 666, 713 / 673, 723 / 676, with a 16-bit
// copy or an unquantized partition 1-6 % at all of them. Below, 2^26 elements 147 / 164, 149 / 150, 148 / 147. Tiles
// filled to 95-98 %: of four waves (buckets of 1184, 2944, 3008, 5952, 6016) 3 * 2^25 elements 219 / 216, 212 / 214,
// 228 / 220, 228 / 220, 221 / 214, 160M 361 / 342, 349 / 330, 347 / 335, 343 / 337, 358 / 342, 300 * 2^20 1-6 % faster;
// of one wave (1472, 1504) 3 * 2^25 206 / 217, 218 / 220, 140 * 2^20 326 / 316, 327 / 318, 160M 356 / 344, 361 / 347,
// 300 * 2^20 641 / 655, 645 / 656. To 92 % (704) 125M 264 / 275, 300 * 2^20 637 / 674, to 81 % (4992) 266 / 287. 4-bit
// codes 125M 252 / 254, 256 / 255, 262 / 250, on a lattice 266 / 265, 270 / 266, 263 / 263. Over tensors, which end
// inside tiles, 200 * 2^20 elements in buckets of 768, five / a hundred to a tensor, 580 / 719, 456 / 487. Without
// codes 125M 241 / 245. code_bits: 0 without codes.
inline bool three_workgroups_stream(int bucket, int buckets, int waves, int rows, uint64_t n, bool tensors,
                                    bool half_gradient, int code_bits, bool lattice) {
    const int filled = waves == 4 || n >= (1ull << 27) ? 95 : 98;
    return rows == 6 && n >= (3ull << 25) && 100 * buckets * (bucket / 32) >= filled * tile_groups(waves, rows) &&
           !tensors && !half_gradient && code_bits == 8 && !lattice;
}

// Workgroups of a learned-level encoder that a compute unit holds at once: by registers (the kernels' launch bounds ask
// for as many) and, for teams of one wave with their tables for each, by LDS. Against five for every shape (us, 4 bit
// coin flip): 134M values in buckets of 608 188 -> 169, 33M in buckets of 2080 93 -> 77.
constexpr int tile_resident(bool coin, int waves, int rows) {
    if (rows <= 4) return 5;
    if (rows == 6) return coin ? 4 : waves == 1 ? 5 : 6;
    return coin ? (waves == 1 ? 3 : 2) : (waves == 1 ? 4 : 5);
}

// ceil(2^18 / bits): slot of the first bit of word w of a tile's code stream = (8 * w * magic) >> 18. A tile has at
// most 2^11 slots, so 8 * w < 2^11 * bits and the product stays below 2^30.
inline uint32_t word_magic(int bits) { return (262144u + (uint32_t)bits - 1u) / (uint32_t)bits; }

}  // namespace qsdp
