// Tile kernel: the encoders and steps for any bucket size (a multiple of 32 up to kMaxBucket) and any code width, both
// run-time values. Serves the bucket sizes the wave kernels are not instantiated for, and tensors too small for them
// with a level table each.
//
// A team of W waves works on a tile of P whole consecutive buckets, i.e. on one contiguous piece of the vector and of
// the code stream: slot s of the tile is its elements 4s .. 4s+3, lane t of the team holds slots r*64W + t of every
// row r, so each load and store instruction of a wave is one contiguous KiB whatever the bucket size, and the values
// stay in registers. A bucket is k = B/32 groups of eight slots. Groups are aligned to eight lanes of a row, so a
// group's minimum and maximum take three DPP steps; the team's 8*W*R group results go through LDS, 2^lanes_log2 lanes
// combine those of one bucket, and the bucket's grid comes back with one 16-byte LDS read per row.
//
// Bound by HBM where a tile is well filled: the step with code output on 125 million parameters in buckets of 768 (W8
// G8) takes 0.266 ms = 6.1 TB/s, against 1.33 ms for a workgroup per bucket that stages its values in LDS and packs
// its codes bit by bit; buckets of 96 on 8 million parameters 0.022 against 0.353 ms. P is the largest count that fits
// (qsdp_tile_plan.hpp, which also says when a tile is smaller), so few slots idle; leaving out the arithmetic of a
// wave's idle rows by branches cost the full tiles 3-10 % (the rows no longer overlap) and won 4 % at the worst fill,
// so it is not done there.
//
// A question that is the same for all rows (whether the tile is contiguous, which grid, eight bits or not) is asked
// once around them: asked in every row or element, as it was, each row was a block of its own that waited for itself.
// us, before / after: eight peers with AdamW 2^26 elements in buckets of 160 / 1504 414 / 371, 454 / 423, four peers
// 156 / 140, 162 / 139, gradient encoder 4 bits, 160, 66.7 / 62.3. Side by side the rows take more registers, so where
// that costs waves which the mode needs, the question stays inside (kAskInside, kAskGridInside, kRowByRow below).
#pragma once

#include "qsdp_params.hpp"
#include "qsdp_levels_kernel.hpp"  // the level tables; widen16
#include "qsdp_tile_plan.hpp"

namespace qsdp {

template <int R, int W>
struct TileLds {
    static constexpr int kTeam = 64 * W;
    static constexpr int kSlots = kTeam * R;
    static constexpr int kGroups = kSlots / 8;
    f4 grid[kGroups];            // per bucket: what its elements need of its grid
    u4 where[kGroups];           // per bucket, tiles that are not contiguous: {offset in the tile, elements, tensor}
    u2 part[kGroups];            // per group: {min, max}
    uint32_t stage[kSlots + 4];  // packed codes: one word of 4 codes per slot, or the tile's code stream
};

template <int W>
__device__ __forceinline__ void team_sync() {
    if constexpr (W == 1) {  // LDS traffic of one wave is processed in order; keep the compiler from reordering it
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// Minimum and maximum over aligned runs of 2^log2 lanes (log2 uniform); all lanes take part.
__device__ __forceinline__ void lanes_minmax(float& lo, float& hi, int log2) {
    if (log2 >= 1) { lo = fminf(lo, dpp_move<0xB1>(lo)); hi = fmaxf(hi, dpp_move<0xB1>(hi)); }
    if (log2 >= 2) { lo = fminf(lo, dpp_move<0x4E>(lo)); hi = fmaxf(hi, dpp_move<0x4E>(hi)); }
    if (log2 >= 3) { lo = fminf(lo, dpp_move<0x141>(lo)); hi = fmaxf(hi, dpp_move<0x141>(hi)); }
    if (log2 >= 4) { lo = fminf(lo, dpp_move<0x140>(lo)); hi = fmaxf(hi, dpp_move<0x140>(hi)); }
    if (log2 >= 5) {
        float a, b;
        swap16(lo, a, b); lo = fminf(a, b);
        swap16(hi, a, b); hi = fmaxf(a, b);
    }
    if (log2 >= 6) {
        float a, b;
        swap32(lo, a, b); lo = fminf(a, b);
        swap32(hi, a, b); hi = fmaxf(a, b);
    }
}

// Code of z among the K = 2^bits levels lv, by the plain definitions: nearest level (ties and
// equal levels: the lowest index) ...
__device__ __forceinline__ uint32_t nearest_level_any(float z, const float* lv, int K) {
    int j = 0;  // ends as the number of levels < z among the first K-1
    for (int step = K >> 1; step >= 1; step >>= 1)
        if (lv[j + step - 1] < z) j += step;
    const int below = j > 0 ? j - 1 : 0;
    int c = fabsf(z - lv[j]) < fabsf(z - lv[below]) ? j : below;
    while (c > 0 && lv[c - 1] == lv[c]) --c;
    return (uint32_t)c;
}

// ... or the coin flip between the two enclosing levels, h the element's 16-bit uniform; z and the levels in units of
// 1/cells.
__device__ __forceinline__ uint32_t stochastic_level_any(float z, float h, const float* lv, int K, float cells) {
    int cnt = 0;  // levels <= z among the first K-1, then the last one
    for (int step = K >> 1; step >= 1; step >>= 1)
        if (lv[cnt + step - 1] <= z) cnt += step;
    if (cnt == K - 1 && lv[K - 1] <= z) ++cnt;
    if (cnt == 0) return 0u;
    const int i = cnt - 1;
    if (i == K - 1) return (uint32_t)i;
    return (uint32_t)i + (coin_up(z, h, level_coin(lv, i, K, cells)) ? 1u : 0u);
}

// The tables of a learned-level encoder for the tensor that a team works on (see qsdp_levels_kernel.hpp), with the
// code width a run-time value: levels and bounds in units of 1/256, a count by cell, by search where the cells are
// crowded. A team takes a run of tiles and sets them up once per tensor. One table, us, against a search and two
// distances per value: 113M values in buckets of 1472, 4 bits 204 -> 116; 27M, 1568, 2 bits 60 -> 29; 125M, 4128, 5
// bits 325 -> 137; coin flip, 125M, 608, 4 bits 229 -> 196. With a table per tensor the tiles that tensors share take
// a pass and a set-up for each (113M 203 -> 120; 33M in 184 tensors, buckets of 96, 81 -> 69).
template <bool COIN>
struct TileLevels {
    static constexpr int C = 256;
    float levels[256];
    float thresholds[COIN ? 1 : 256];
    LevelCoin coin[COIN ? 256 : 1];
    LevelCell cells[C + 1];
};

// What the launch adds to Params: the number of tiles (a 64-bit division in every wave's prologue otherwise), the
// tile's shape (see TilePlan) and ceil(2^18 / width) of the stored codes.
struct TileArgs {
    uint64_t tiles;
    int buckets, lanes_log2;
    uint32_t group_magic, word_magic;
};

// Workgroups to a compute unit that a kernel's registers must allow (1: what the compiler makes of it). The receive side
// with AdamW fits four of them into 128 registers without spilling where it has up to four rows, and needs more if left
// alone. us, left alone / four: eight peers, 2^25 elements in buckets of 96, 416, 800, 3488 202 / 194, 203 / 192, 197 /
// 190, 209 / 195, two peers, 2^26 316 / 306, 304 / 302, 306 / 311, 319 / 303; 2^18, eight peers, 9.5 / 9.4, 9.5 / 9.4,
// 10.5 / 10.4, 15.6 / 15.9.
constexpr int tile_min_blocks(int mode, int waves, int rows) {
    if (mode_is_levels(mode)) return tile_resident(mode == MODE_LEVELS_COIN, waves, rows);
    if (mode == MODE_RECV_ADAMW && rows <= 4) return 4;
    return 1;
}

template <int MODE, int R, int W>
__global__ void __launch_bounds__(256, tile_min_blocks(MODE, W, R))
    tile_kernel(const Params args, const Segment* __restrict__ segs, const TileArgs a) {
    static_assert(R % 2 == 0 && R <= kTileMaxRows && (W == 1 || W == 4), "shape");
    typedef TileLds<R, W> Lds;
    constexpr int TEAM = Lds::kTeam;
    constexpr bool kWritesX = MODE == MODE_FUSED || MODE == MODE_ADAMW || mode_is_recv(MODE);
    constexpr bool kLevels = mode_is_levels(MODE);
    // Eight rows of the weight encoder one after the other: side by side they take 105 registers instead of 64, four
    // waves to a SIMD instead of seven (us, 2^26 elements in buckets of 2080 / 7200: 4 bits 54.7 / 53.6 and side by
    // side 60.4 / 58.1, on a lattice 59.4 / 55.8 and 70.7 / 66.1; 8 bits 58.5 / 58.3 and, packed by the converting
    // instruction, 56.6 / 56.5, which does not make up for the others).
    constexpr bool kRowByRow = MODE == MODE_WEIGHT && R == 8;
    // A call's last tile, which its buckets seldom fill, runs the instructions of all others in the shapes that small
    // calls get: what a single wave runs comes from memory, line after line, and such a call waits for it (us, 65571
    // elements in buckets of 320 / 2336, on a path of its own / with the others: AdamW step 8.5 / 7.2, 9.9 / 7.2, step
    // 5.2 / 4.6, 7.3 / 5.9, gradient encoder 3.8 / 3.3, 5.0 / 4.0, four peers 5.2 / 4.8, 7.5 / 5.9; 3M, 768, step 10.6
    // / 9.0). Large calls do not: there a team of one wave and, where the patches take registers, the weight encoder
    // and the steps of eight rows were 2-5 % slower (100M, 2336, AdamW step 492 / 514), and so was the gradient encoder of
    // six and eight rows (125M, 4 bits, buckets of 2080 / 4128: 111.0 / 120.4 on a path of its own, 113.7 / 124.2).
    constexpr bool kTailsInline =
        R == 2 || (W == 4 && MODE != MODE_WEIGHT && !(R == 8 && (MODE == MODE_FUSED || MODE == MODE_ADAMW)) &&
                   !(R > 4 && MODE == MODE_GRAD));
    // The parameters are read again for every tile, and again for its weights, and the keys of the ten rounds are
    // computed for every block: held across the loop they were 50-150 scalar registers too many, each written to and
    // read from a lane of a vector register (step, four rows, 77 -> 24, and 90 -> 87 vector registers). 216 calls of
    // 2^16 to 10^8 elements in buckets of 96 to 2336: code-resident step 1.05-1.08 times faster, receive side
    // 1.02-1.07, steps 1.02-1.04; the weight encoder's larger tiles and the nearest level, with ten, lost 0-2 %. The
    // gradient encoder, whose keys alone are computed again, waits for the parameters before its loads: buckets of 32
    // to 2016, read once against again, 1.01-1.04 times faster on 10^6 to 8*10^6 values that are not in the caches (8M
    // in buckets of 1504, 13.1 -> 12.3 us, seven waves to a SIMD instead of six) and on 65571 ones, cached 0.98-1.03,
    // large ones 0.99-1.02.
    constexpr bool kReadAgain = MODE != MODE_LEVELS && MODE != MODE_GRAD && (MODE != MODE_WEIGHT || R == 2);
    // The first team takes the call's last tile, which takes longer for its short bucket, and the last team the first;
    // all others keep theirs, so that a tile meets its codes in the same L2 as in the next call. us, each its own / so,
    // buckets of 768, 1504, 2336: 5M elements, step 12.7 / 11.7, 13.0 / 11.9, 14.7 / 12.8, AdamW step 35.8 / 31.0,
    // 33.0 / 30.9, 36.8 / 31.1, four peers 16.0 / 15.3, 16.2 / 15.5, 18.5 / 18.4; from 20M on 0-2 %. The weight encoder
    // was slower (12M, 32, 18.0 / 19.5), two rows gained nothing below 3M.
    constexpr bool kLastFirst = !kLevels && MODE != MODE_WEIGHT && R > 2;
    __shared__ Lds lds_all[4 / W];
    constexpr bool kCoin = MODE == MODE_LEVELS_COIN;
    __shared__ char level_lds[kLevels ? 4 / W * sizeof(TileLevels<kCoin>) : 1] __attribute__((aligned(16)));
    const uint32_t wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tid = W == 1 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
    Lds& lds = lds_all[W == 1 ? wave_in_block : 0];
    TileLevels<kCoin>& lt = reinterpret_cast<TileLevels<kCoin>*>(level_lds)[W == 1 && kLevels ? wave_in_block : 0];
    uint32_t loaded_tensor = ~0u;  // whose level table the team holds
    bool level_by_cell = false;    // ... and how it is used

    const int B = args.bucket;
    const int k = B >> 5;      // groups of a bucket
    const int S = B >> 2;      // slots of a bucket
    const int P = a.buckets;   // buckets of a full tile
    const PhiloxKey key = launch_key<MODE>(args);
    const Shifts shifts = launch_shifts<MODE, false, MODE == MODE_WEIGHT && R == 4>(args, key);
    uint32_t saturated = 0;

    uint64_t unit0 = W == 1 ? (uint64_t)blockIdx.x * 4u + wave_in_block : blockIdx.x;
    uint64_t unit_stride = W == 1 ? (uint64_t)gridDim.x * 4u : gridDim.x;
    uint64_t unit_end = a.tiles;
    if constexpr (kLevels) {  // a run of tiles: the tables are set up once per tensor and run
        const uint64_t run = (a.tiles + unit_stride - 1) / unit_stride;
        unit0 *= run;
        unit_end = unit0 + run < a.tiles ? unit0 + run : a.tiles;
        unit_stride = 1;
    }
    // row r of this lane: its slot; bucket of a slot in the tile
    auto slot_of = [&](int r) { return r * TEAM + tid; };
    auto bucket_of_slot = [&](int slot) { return (int)(((uint32_t)slot >> 3) * a.group_magic >> 16); };

    for (uint64_t next = unit0; next < unit_end; next += unit_stride) {
        const uint64_t unit = !kLastFirst ? next : next == 0 ? unit_end - 1 : next == unit_end - 1 ? 0 : next;
        // keeps what follows from the lane's number alone (slots, buckets, offsets of every row) out of registers that
        // live across the loop
        asm volatile("" : "+v"(tid));
        Params p = kReadAgain ? params_again() : args;
        const float Lg = (float)((1 << p.gbits) - 1);
        const uint32_t top16_g = (uint32_t)((1 << p.gbits) - 1) << 16;
        const bool grad_shift = (p.flags & FLAG_GRAD_SHIFT) != 0;
        const int odd = tid & 1;
        const uint64_t bucket0 = unit * (uint64_t)P;
        const uint64_t left = p.num_buckets - bucket0;
        const int here = left < (uint64_t)P ? (int)left : P;  // buckets of this tile
        const BucketRef first = locate_bucket(p, segs, bucket0, bucket0, (uint32_t)B);
        const uint64_t e0 = first.e0;
        // Contiguous: one piece of one tensor; full buckets or, where tails run with the others, a slot at least.
        const bool whole = kTailsInline ? first.left > (uint64_t)(here - 1) * (uint64_t)B && first.left >= 4u
                                        : here == P && first.left >= (uint64_t)P * (uint64_t)B;
        const uint64_t word0 = bucket0 * (uint64_t)(B >> 5);  // times the code width: the tile's first code word
        const int used = here * S;                            // slots of these buckets
        // of a contiguous tile: its elements, the slots that exist in full, the elements of the one after them
        const int existing = kTailsInline && first.left < (uint64_t)(4 * used) ? (int)first.left : 4 * used;
        const int full = kTailsInline ? existing >> 2 : used;
        const int partial = kTailsInline ? existing & 3 : 0;
        const bool ragged = kTailsInline ? !whole || full != used : !whole;
        // whether the row is computed: the smallest teams leave an unused second one out
        auto computed = [&](int r) { return R > 2 || r == 0 || used > TEAM; };
        if (W > 1) team_sync<W>();  // the previous tile's LDS reads are done
        if (__builtin_expect(!whole, 0)) {
            if (tid < P) {
                u4 w = {0u, 0u, 0u, 0u};
                if (tid < here) {
                    const BucketRef ref = locate_bucket(p, segs, bucket0, bucket0 + (uint64_t)tid, (uint32_t)B);
                    w[0] = (uint32_t)(ref.e0 - e0);
                    w[1] = ref.m;
                    w[2] = ref.tensor;
                }
                lds.where[tid] = w;
            }
            team_sync<W>();
        }
        // Offset from e0 of the first element of a slot, and how many of its four elements exist, in a tile that is
        // not contiguous.
        struct Place { uint32_t rel; int count; };
        auto place = [&](int slot) -> Place {
            asm volatile("" : "+v"(slot));  // not worth keeping for the unlikely path
            const int b = bucket_of_slot(slot);
            if (b >= here) return {0u, 0};
            const u4 w = lds.where[b];
            const int off = (slot - b * S) * 4;
            const int c = (int)w[1] - off;
            return {w[0] + (uint32_t)off, c < 0 ? 0 : c > 4 ? 4 : c};
        };
        // In a contiguous one slot s is elements 4s .. 4s+3; the slots past the last full one read the tile's first
        // elements instead: in bounds, and their values go nowhere. So a call's last tile runs the instructions of all
        // others, and its own are only the patches of the slot that exists in part.
        auto patch = [&](const float* base, float (&v)[R][4]) {  // once the tile's loads are under way
            if (kTailsInline && __builtin_expect(whole && partial != 0, 0)) {
                const float* from = base + e0 + 4 * full;
                const float x0 = from[0], x1 = partial > 1 ? from[1] : 0.0f, x2 = partial > 2 ? from[2] : 0.0f;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool mine = slot_of(r) == full;
                    v[r][0] = mine ? x0 : v[r][0];
                    v[r][1] = mine ? x1 : v[r][1];
                    v[r][2] = mine ? x2 : v[r][2];
                }
            }
        };
        auto load = [&](const float* base, float (&v)[R][4]) {
            const char* at = reinterpret_cast<const char*>(base + e0);
            if (__builtin_expect(whole, 1)) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t s = slot_of(r) < full ? (uint32_t)slot_of(r) : 0u;
                    const f4 x = __builtin_nontemporal_load(reinterpret_cast<const f4*>(at + s * 16u));
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[r][i] = x[i];
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const Place s = place(slot_of(r));
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[r][i] = i < s.count ? (base + e0 + s.rel)[i] : 0.0f;
                }
            }
        };
        // 16-bit values are two to a word in the first two places of a slot until they are widened: at once, since with
        // a patch in between the compiler keeps both for the steps (four waves, eight rows: 175 registers instead of
        // 156); but after it in the gradient encoder, which would keep the widened ones for longer (102 against 89).
        constexpr bool kWidenLater = kTailsInline && MODE == MODE_GRAD;
        auto widen = [&](bool bf16, float (&v)[R][4]) {
            auto all = [&](auto widened) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t h[2] = {__float_as_uint(v[r][0]), __float_as_uint(v[r][1])};
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[r][i] = widened(i & 1 ? h[i >> 1] >> 16 : h[i >> 1] & 0xFFFFu);
                }
            };
            if (bf16) all([](uint32_t h) { return widen16<true>(h); });
            else all([](uint32_t h) { return widen16<false>(h); });
        };
        auto load_half = [&](const void* base, bool bf16, float (&v)[R][4]) {
            const uint16_t* first_half = static_cast<const uint16_t*>(base) + e0;
            uint32_t h[R][2];
            if (__builtin_expect(whole, 1)) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t s = slot_of(r) < full ? (uint32_t)slot_of(r) : 0u;
                    const u2 x = __builtin_nontemporal_load(
                        reinterpret_cast<const u2*>(reinterpret_cast<const char*>(first_half) + s * 8u));
                    h[r][0] = x[0];
                    h[r][1] = x[1];
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const Place s = place(slot_of(r));
                    h[r][0] = h[r][1] = 0u;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (i < s.count) h[r][i >> 1] |= (uint32_t)first_half[s.rel + i] << (16 * (i & 1));
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 2; ++i) v[r][i] = __uint_as_float(h[r][i]);
            if (!kWidenLater) widen(bf16, v);
        };
        auto patch_half = [&](const void* base, bool bf16, float (&v)[R][4]) {
            if (kTailsInline && __builtin_expect(whole && partial != 0, 0)) {
                const uint16_t* from = static_cast<const uint16_t*>(base) + e0 + 4 * full;
                const uint32_t h[3] = {from[0], partial > 1 ? from[1] : 0u, partial > 2 ? from[2] : 0u};
                float x[3];
                if (kWidenLater) {
                    x[0] = __uint_as_float(h[0] | (h[1] << 16));
                    x[1] = __uint_as_float(h[2]);
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i) x[i] = bf16 ? widen16<true>(h[i]) : widen16<false>(h[i]);
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int i = 0; i < (kWidenLater ? 2 : 3); ++i) v[r][i] = slot_of(r) == full ? x[i] : v[r][i];
            }
            if (kWidenLater) widen(bf16, v);
        };
        auto store = [&](float* base, const float (&v)[R][4]) {
            char* at = reinterpret_cast<char*>(base + e0);
            if (__builtin_expect(whole, 1)) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const f4 x = {v[r][0], v[r][1], v[r][2], v[r][3]};
                    if (slot_of(r) < full)
                        __builtin_nontemporal_store(x, reinterpret_cast<f4*>(at + (uint32_t)slot_of(r) * 16u));
                }
                if (kTailsInline && __builtin_expect(partial != 0, 0)) {
                    float x[3] = {};
                    bool any = false;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const bool mine = slot_of(r) == full;
                        any |= mine;
#pragma unroll
                        for (int i = 0; i < 3; ++i) x[i] = mine ? v[r][i] : x[i];
                    }
                    float* to = base + e0 + 4 * full;
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (any && i < partial) to[i] = x[i];
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const Place s = place(slot_of(r));
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (i < s.count) (base + e0 + s.rel)[i] = v[r][i];
                }
            }
        };
        auto store_half = [&](void* base, bool f16, const float (&v)[R][4]) {
            uint16_t* first_half = static_cast<uint16_t*>(base) + e0;
            if (__builtin_expect(whole, 1)) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const u2 x = {half_bits(v[r][0], f16) | (half_bits(v[r][1], f16) << 16),
                                  half_bits(v[r][2], f16) | (half_bits(v[r][3], f16) << 16)};
                    if (slot_of(r) < full)
                        __builtin_nontemporal_store(
                            x, reinterpret_cast<u2*>(reinterpret_cast<char*>(first_half) + (uint32_t)slot_of(r) * 8u));
                }
                if (kTailsInline && __builtin_expect(partial != 0, 0)) {
                    float x[3] = {};
                    bool any = false;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const bool mine = slot_of(r) == full;
                        any |= mine;
#pragma unroll
                        for (int i = 0; i < 3; ++i) x[i] = mine ? v[r][i] : x[i];
                    }
                    uint16_t* to = first_half + 4 * full;
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (any && i < partial) to[i] = (uint16_t)half_bits(x[i], f16);
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const Place s = place(slot_of(r));
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (i < s.count) first_half[s.rel + i] = (uint16_t)half_bits(v[r][i], f16);
                }
            }
        };
        // Rounding uniforms of rows 2cp and 2cp + 1: the pair's even lane draws the block of the first, its odd lane
        // that of the second.
        uint32_t block_rel[R / 2];
        auto locate_blocks = [&]() {
#pragma unroll
            for (int cp = 0; cp < R / 2; ++cp) block_rel[cp] = (uint32_t)((2 * cp + odd) * TEAM + tid - odd) >> 1;
            if (__builtin_expect(!whole, 0)) {
#pragma unroll
                for (int cp = 0; cp < R / 2; ++cp) block_rel[cp] = place((2 * cp + odd) * TEAM + tid - odd).rel >> 3;
            }
        };
        auto uniforms = [&](int cp, uint32_t (&h)[4]) {
            uint32_t k0 = key.k0, k1 = key.k1;
            asm volatile("" : "+s"(k0), "+s"(k1));
            uniforms_of_pair<(MODE == MODE_GRAD || MODE == MODE_LEVELS_COIN)>(p.block0 + (e0 >> 3) + block_rel[cp], odd,
                                                                              k0, k1, h);
        };
        // Minimum and maximum of every bucket of the tile, then its grid: make(lo, hi, bucket in the tile) in the
        // lanes that combine that bucket, the result in lds.grid for all.
        auto bucket_grids = [&](const float (&v)[R][4], auto make) {
            float row_lo[R], row_hi[R];
            auto range = [&](int r) {
                row_lo[r] = fminf(fminf(v[r][0], v[r][1]), fminf(v[r][2], v[r][3]));
                row_hi[r] = fmaxf(fmaxf(v[r][0], v[r][1]), fmaxf(v[r][2], v[r][3]));
            };
            auto range_of_existing = [&](int r) {
                const int c = kTailsInline && whole ? existing - 4 * slot_of(r) : place(slot_of(r)).count;
                row_lo[r] = __builtin_inff();
                row_hi[r] = -__builtin_inff();
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    row_lo[r] = i < c ? fminf(row_lo[r], v[r][i]) : row_lo[r];
                    row_hi[r] = i < c ? fmaxf(row_hi[r], v[r][i]) : row_hi[r];
                }
            };
            auto over_group = [&](int r) {
                row_lo[r] = group_min<8>(row_lo[r]);
                row_hi[r] = group_max<8>(row_hi[r]);
            };
            auto keep = [&](int r) {
                const u2 e = {__float_as_uint(row_lo[r]), __float_as_uint(row_hi[r])};
                lds.part[slot_of(r) >> 3] = e;
            };
            if constexpr (kRowByRow) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    range(r);
                    if (__builtin_expect(ragged, 0)) range_of_existing(r);
                    over_group(r);
                    if ((tid & 7) == 0) keep(r);
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) range(r);
                if (__builtin_expect(ragged, 0)) {
#pragma unroll
                    for (int r = 0; r < R; ++r) range_of_existing(r);
                }
#pragma unroll
                for (int r = 0; r < R; ++r) over_group(r);
                if ((tid & 7) == 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r) keep(r);
                }
            }
            team_sync<W>();
            const int b = tid >> a.lanes_log2;
            float lo = __builtin_inff(), hi = -__builtin_inff();
            if (b < here)
                for (int i = tid & ((1 << a.lanes_log2) - 1); i < k; i += 1 << a.lanes_log2) {
                    const u2 e = lds.part[b * k + i];
                    lo = fminf(lo, __uint_as_float(e[0]));
                    hi = fmaxf(hi, __uint_as_float(e[1]));
                }
            lanes_minmax(lo, hi, a.lanes_log2);
            const f4 g = make(lo, hi, b);
            if (b < here && (tid & ((1 << a.lanes_log2) - 1)) == 0) lds.grid[b] = g;
            team_sync<W>();
        };
        auto first_of_bucket = [&](int b) { return b < here && (tid & ((1 << a.lanes_log2) - 1)) == 0; };
        auto write_meta = [&](int b, float base, float scale) {
            if (first_of_bucket(b)) {
                const u2 m = {__float_as_uint(base), __float_as_uint(scale)};
                *reinterpret_cast<u2*>(p.meta + 2 * (bucket0 + (uint64_t)b)) = m;
            }
        };
        // The `bits` wide codes of the tile: words of the code stream that starts at `words`, fetched now ...
        auto fetch_words = [&](const uint32_t* words, int bits, uint32_t (&w)[R]) {
            const int total = used * bits >> 3;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = slot_of(r);
                w[r] = i < total ? __builtin_nontemporal_load(words + i) : 0u;
            }
        };
        // ... and taken apart: the four codes of each of the lane's slots. The stage holds no other words then.
        auto unpack = [&](const uint32_t (&w)[R], int bits, float (&c)[R][4]) {
            if (bits != 8) {  // at 8 bits word s is slot s
                team_sync<W>();
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (r * 8 < R * bits) lds.stage[slot_of(r)] = w[r];
                team_sync<W>();
            }
            uint32_t q[R];
#pragma unroll
            for (int r = 0; r < R; ++r) q[r] = w[r];
            if (bits != 8) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t bit = (uint32_t)(slot_of(r) * 4 * bits);
                    const uint64_t two = (uint64_t)lds.stage[bit >> 5] | ((uint64_t)lds.stage[(bit >> 5) + 1] << 32);
                    q[r] = (uint32_t)(two >> (bit & 31u));
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    c[r][i] = (float)__builtin_amdgcn_ubfe(q[r], (uint32_t)(i * bits), (uint32_t)bits);
        };
        // The reverse: pack the codes and write the tile's part of the code stream. Slots past a short bucket's end
        // carry zeros.
        auto store_packed = [&](uint32_t (&q)[R], int bits) {
            uint32_t* out = p.codes + word0 * (uint64_t)bits;
            if (__builtin_expect(!whole, 0)) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int c = place(slot_of(r)).count;
                    if (c < 4) q[r] &= (1u << (c * bits)) - 1u;
                }
            } else if (kTailsInline && __builtin_expect(full != used, 0)) {
                const uint32_t some = (1u << (partial * bits)) - 1u;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t past = slot_of(r) == full ? some : 0u;
                    q[r] &= slot_of(r) < full ? ~0u : past;
                }
            }
            if (bits == 8) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (slot_of(r) < used) __builtin_nontemporal_store(q[r], out + slot_of(r));
                return;
            }
            team_sync<W>();
#pragma unroll
            for (int r = 0; r < R; ++r) lds.stage[slot_of(r)] = q[r];
            team_sync<W>();
            const int total = used * bits >> 3;
            for (int w = tid; w < total; w += TEAM) {
                int s = (int)((uint32_t)(8 * w) * a.word_magic >> 18);  // slot of the word's first bit
                int at = s * 4 * bits - 32 * w;                         // where its codes start: at or before bit 0
                uint32_t word = lds.stage[s] >> -at;
                for (at += 4 * bits; at < 32; at += 4 * bits) word |= lds.stage[++s] << at;
                __builtin_nontemporal_store(word, out + w);
            }
        };
        auto store_words = [&](const uint32_t (&code)[R][4], int bits) {
            uint32_t q[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                q[r] = code[r][0] | (code[r][1] << bits);
                q[r] |= (code[r][2] << (2 * bits)) | (code[r][3] << (3 * bits));
            }
            store_packed(q, bits);
        };

        float w[R][4];  // the values that get weight-quantized
        if constexpr (mode_local_gradient(MODE)) {
            float gv[R][4];
            float mom[R][4], var[R][4];  // AdamW modes only
            uint32_t old_words[R];       // code-resident modes only
            if constexpr (mode_codes_resident(MODE))
                fetch_words(p.codes + word0 * (uint64_t)p.wbits, p.wbits, old_words);
            if (mode_mixed_precision(MODE) && p.g_half != 0u) load_half(p.g, p.g_half == 1u, gv);
            else load(p.g, gv);
            if constexpr (MODE == MODE_FUSED || MODE == MODE_ADAMW) load(p.x, w);
            if constexpr (mode_local_adamw(MODE)) {
                load(p.mom, mom);
                load(p.var, var);
            }
            if (mode_mixed_precision(MODE) && p.g_half != 0u) patch_half(p.g, p.g_half == 1u, gv);
            else patch(p.g, gv);
            if constexpr (MODE == MODE_FUSED || MODE == MODE_ADAMW) patch(p.x, w);
            if constexpr (mode_local_adamw(MODE)) {
                patch(p.mom, mom);
                patch(p.var, var);
            }
            if constexpr (mode_codes_resident(MODE)) {
                unpack(old_words, p.wbits, w);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int b = bucket_of_slot(slot_of(r));
                    const float* m = p.meta + 2 * (bucket0 + (uint64_t)(b < here ? b : 0));
                    const float base = m[0], scale = m[1];
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[r][i] = fmaf(w[r][i], scale, base);
                }
            }
            bucket_grids(gv, [&](float lo, float hi, int b) -> f4 {
                const MinMaxGrid g = make_minmax_grid(lo, hi, Lg, (p.flags & FLAG_SYMMETRIC) != 0);
                const float base = grad_shift ? fmaf(shifts.xi_g, g.scale, g.lo) : g.lo;
                if constexpr (MODE == MODE_GRAD) write_meta(b, base, g.scale);
                return f4{g.lo, g.inv, g.scale, base};
            });
            uint32_t code[MODE == MODE_GRAD ? R : 1][4] = {};
            auto grid_of_row = [&](int r) -> f4 { return lds.grid[bucket_of_slot(slot_of(r))]; };
            // The question outside the rows, so that these are straight-line code (gradient encoder, 2^26 elements
            // from bf16, 3 bits, buckets of 160: 68.7 -> 65.7 us). The steps on resident weights ask it for every
            // element: with the rows of their divisions side by side AdamW's take 40 more registers (2^26 elements,
            // buckets of 1504, 333 against 351 us), the code-resident step's 20-30 (four rows: 92 for 73, five waves to
            // a SIMD instead of six; us, 125M in buckets of 608 / 800 / 2080 / 3488, 8 bits 157 / 167 / 190 / 181
            // against 164 / 182 / 208 / 194, 5 bits 176 / 186 / 226 / 208 against 189 / 202 / 242 / 225), and the plain
            // step is bound by memory and 1-2 % slower.
            constexpr bool kAskInside = MODE == MODE_FUSED || mode_codes_resident(MODE) || mode_local_adamw(MODE);
            if (!kAskInside && grad_shift) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (!computed(r)) continue;
                    const f4 gr = grid_of_row(r);
                    const MinMaxGrid grid = {gr[0], gr[2], gr[1]};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float c = weight_code_minmax(gv[r][i], grid, Lg, shifts.xi_g);
                        if constexpr (MODE == MODE_GRAD) code[r][i] = (uint32_t)c;
                        else
                            w[r][i] = step_value<MODE>(p, w[r][i], fmaf(c, grid.scale, gr[3]), mom[r][i], var[r][i]);
                    }
                }
            } else {
                locate_blocks();
#pragma unroll
                for (int cp = 0; cp < R / 2; ++cp) {
                    uint32_t h[4] = {0u, 0u, 0u, 0u};
                    if (!kAskInside || !grad_shift) uniforms(cp, h);
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int r = 2 * cp + half;
                        if (!computed(r)) continue;
                        const f4 gr = grid_of_row(r);
                        const MinMaxGrid grid = {gr[0], gr[2], gr[1]};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t u = uniform16(h, 4 * half + i);
                            if constexpr (MODE == MODE_GRAD) {
                                code[r][i] = grad_code_int(gv[r][i], grid, top16_g, u);
                            } else {
                                const float c = kAskInside && grad_shift
                                                    ? weight_code_minmax(gv[r][i], grid, Lg, shifts.xi_g)
                                                    : grad_code(gv[r][i], grid, top16_g, u);
                                w[r][i] =
                                    step_value<MODE>(p, w[r][i], fmaf(c, grid.scale, gr[3]), mom[r][i], var[r][i]);
                            }
                        }
                    }
                }
            }
            if constexpr (mode_local_adamw(MODE)) {
                store(p.mom, mom);
                store(p.var, var);
            }
            if constexpr (MODE == MODE_GRAD) {
                store_words(code, p.gbits);
                continue;
            }
        } else if constexpr (mode_is_recv(MODE)) {
            load(p.x, w);
            float mom[R][4], var[R][4];  // MODE_RECV_ADAMW only
            if constexpr (MODE == MODE_RECV_ADAMW) {
                load(p.mom, mom);
                load(p.var, var);
            }
            // ghat = alpha * (((d_0 + d_1) + d_2) + ...), the words of two peers in flight at a time
            float sum[R][4];
            const uint32_t* words = p.peer_codes + word0 * (uint64_t)p.gbits;
            for (int peer0 = 0; peer0 < p.npeers; peer0 += 2) {
                const bool two = peer0 + 1 < p.npeers;
                const uint64_t next = two ? peer0 + 1 : peer0;  // past the last peer: read that one again, in bounds
                uint32_t words_a[R], words_b[R];
                fetch_words(words + (uint64_t)peer0 * p.peer_codes_stride_words, p.gbits, words_a);
                fetch_words(words + next * p.peer_codes_stride_words, p.gbits, words_b);
                f4 meta = {0.0f, 0.0f, 0.0f, 0.0f};
                if (tid < here) {
                    const float* meta0 = p.peer_meta + 2 * (bucket0 + (uint64_t)tid);
                    const float* m = meta0 + (uint64_t)peer0 * p.peer_meta_stride_floats;
                    const float* m2 = meta0 + next * p.peer_meta_stride_floats;
                    meta = f4{m[0], m[1], m2[0], m2[1]};
                }
                team_sync<W>();  // the previous pair's meta has been read
                if (tid < here) lds.grid[tid] = meta;
                float c[R][4];
                unpack(words_a, p.gbits, c);
                team_sync<W>();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const f4 m = lds.grid[bucket_of_slot(slot_of(r))];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float d = fmaf(c[r][i], m[1], m[0]);
                        sum[r][i] = peer0 == 0 ? d : sum[r][i] + d;
                    }
                }
                if (two) {
                    unpack(words_b, p.gbits, c);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const f4 m = lds.grid[bucket_of_slot(slot_of(r))];
#pragma unroll
                        for (int i = 0; i < 4; ++i) sum[r][i] = sum[r][i] + fmaf(c[r][i], m[3], m[2]);
                    }
                }
            }
            patch(p.x, w);
            if constexpr (MODE == MODE_RECV_ADAMW) {
                patch(p.mom, mom);
                patch(p.var, var);
            }
            team_sync<W>();
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (computed(r)) w[r][i] = step_value<MODE>(p, w[r][i], p.alpha * sum[r][i], mom[r][i], var[r][i]);
            if constexpr (MODE == MODE_RECV_ADAMW) {
                store(p.mom, mom);
                store(p.var, var);
            }
        } else {
            load(p.xin, w);
            patch(p.xin, w);
        }

        if (kReadAgain) p = params_again();
        const float Lw = (float)((1 << p.wbits) - 1);
        const Divider div = {p.delta, p.inv_delta, p.delta_pow2 != 0};
        const bool lattice = p.delta > 0.0f;
        const bool keep_master = kWritesX && (p.flags & FLAG_KEEP_MASTER) != 0;
        const float xi = shifts.xi;
        // the full-precision partition keeps the updated value itself
        if (kWritesX && keep_master) store(p.x, w);

        uint32_t code[R][4] = {};
        if constexpr (kLevels) {
            const int K = 1 << p.wbits;
            constexpr int C = TileLevels<kCoin>::C;
            bucket_grids(w, [&](float lo, float hi, int b) -> f4 {
                const MinMaxGrid g = make_minmax_grid(lo, hi, 1.0f, false);
                write_meta(b, g.lo, g.scale);
                return f4{g.lo, g.inv * (float)C, 0.0f, 0.0f};
            });
            // One pass per tensor of the tile (one for nearly all): its tables come into LDS, its buckets keep their
            // codes.
            uint32_t tensor = p.levels_per_tensor != 0u ? first.tensor : 0u, last_tensor = tensor;
            if (__builtin_expect(!whole, 0) && p.levels_per_tensor != 0u)
                last_tensor = __builtin_amdgcn_readfirstlane(lds.where[here - 1][2]);
            const bool single = tensor == last_tensor;
            for (;; ++tensor) {
                // keeps values and uniforms of all rows from being held across the passes
                asm volatile("" : "+v"(tid));
                if (tensor != loaded_tensor) {
                    auto any = [](bool c) -> bool {
                        if constexpr (W == 1) {
                            team_sync<W>();
                            return __builtin_amdgcn_ballot_w64(c) != 0;
                        } else {
                            return __syncthreads_or(c) != 0;
                        }
                    };
                    team_sync<W>();
                    for (int i = tid; i < K; i += TEAM) lt.levels[i] = p.levels[(uint64_t)tensor * K + i] * (float)C;
                    team_sync<W>();
                    uint32_t found = 0;
                    if constexpr (kCoin) {
                        for (int i = tid; i < K; i += TEAM) lt.coin[i] = level_coin(lt.levels, i, K, (float)C);
                    } else {
                        for (int i = tid; i < K - 1; i += TEAM)
                            if (!level_threshold(lt.levels, i, K, (float)C, lt.thresholds + i)) found |= LEVELS_UNUSABLE;
                        team_sync<W>();
                    }
                    found |= fill_level_cells<C, TEAM>(lt.cells, kCoin ? lt.levels + 1 : lt.thresholds, K, tid);
                    level_by_cell = !any((found & (LEVELS_UNUSABLE | LEVELS_CROWDED)) != 0);
                    loaded_tensor = tensor;
                }
                // by cell, by search and by search for some of the buckets are loops of their own, so that each is
                // straight-line code over the rows
                if constexpr (kCoin) locate_blocks();
                auto encode = [&](auto mine, auto code_of) {
#pragma unroll
                    for (int cp = 0; cp < R / 2; ++cp) {
                        uint32_t h[4] = {0u, 0u, 0u, 0u};
                        if constexpr (kCoin) uniforms(cp, h);
#pragma unroll
                        for (int half = 0; half < 2; ++half) {
                            const int r = 2 * cp + half;
                            if (!computed(r)) continue;
                            const int b = bucket_of_slot(slot_of(r));
                            const f4 gr = lds.grid[b];
                            if (mine(b)) {
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    code[r][i] = code_of((w[r][i] - gr[0]) * gr[1], (float)uniform16(h, 4 * half + i));
                            }
                        }
                    }
                };
                auto every = [](int) { return true; };
                auto search = [&](float z, float h) -> uint32_t {
                    return kCoin ? stochastic_level_any(z, h, lt.levels, K, (float)C)
                                 : nearest_level_any(z, lt.levels, K);
                };
                auto lookup = [&](float z, float h) -> uint32_t {
                    const uint32_t c = (uint32_t)z;
                    const LevelCell e = lt.cells[c < (uint32_t)C ? c : (uint32_t)C];
                    const uint32_t n = (e.count & 0xFFFFu) + (e.next <= z ? (e.count >> 16) + 1u : 0u);
                    if constexpr (!kCoin) return n;
                    return n + (coin_up(z, h, lt.coin[n]) ? 1u : 0u);
                };
                if (__builtin_expect(single && level_by_cell, 1)) {
                    encode(every, lookup);
                    break;
                }
                if (single) {
                    encode(every, search);
                    break;
                }
                encode([&](int b) { return b < here && lds.where[b][2] == tensor; },
                       [&](float z, float h) {  // the coin flip's lookup would cost this path too many registers
                           return !kCoin && level_by_cell ? lookup(z, h) : search(z, h);
                       });
                if (tensor == last_tensor) break;
            }
            store_words(code, p.wbits);
            continue;
        }

        const bool emit = MODE == MODE_WEIGHT || mode_codes_resident(MODE) || p.codes != nullptr;
        bucket_grids(w, [&](float lo, float hi, int b) -> f4 {
            float base, scale, origin, inv = 0.0f;
            if (lattice) {
                lo = lo + 0.0f;
                origin = rintf(div_delta(lo, div) - xi);
                base = (origin + xi) * p.delta;
                scale = p.delta;
            } else {
                const MinMaxGrid g = make_minmax_grid(lo, hi, Lw, (p.flags & FLAG_SYMMETRIC) != 0);
                base = fmaf(xi, g.scale, g.lo);
                scale = g.scale;
                origin = g.lo;
                inv = g.inv;
            }
            if (emit) write_meta(b, base, scale);
            return f4{origin, inv, scale, base};
        });
        const bool want16 = (MODE == MODE_FUSED || MODE == MODE_ADAMW) && p.x16 != nullptr;
        auto weight_grid = [&](int r) -> f4 { return lds.grid[bucket_of_slot(slot_of(r))]; };
        auto onto_lattice = [&](int r) {
            const f4 gr = weight_grid(r);
            const int n = __builtin_expect(whole, 1) ? existing - 4 * slot_of(r) : place(slot_of(r)).count;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t over = 0;
                const float c = weight_code_lattice(w[r][i], div, xi, gr[0], Lw, over);
                saturated += i < n ? over : 0u;
                code[r][i] = (uint32_t)c;
                w[r][i] = fmaf(c, gr[2], gr[3]);
            }
        };
        auto onto_minmax = [&](int r) {
            const f4 gr = weight_grid(r);
            const MinMaxGrid grid = {gr[0], gr[2], gr[1]};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float c = weight_code_minmax(w[r][i], grid, Lw, xi);
                code[r][i] = (uint32_t)c;
                w[r][i] = fmaf(c, gr[2], gr[3]);
            }
        };
        // Which grid is a question for every row in the weight encoder's large tiles, whose divisions by delta would
        // cost waves side by side (4 bits, 2^26 elements in buckets of 288 / 1504, 54.9 / 54.1 against 57.9 / 56.6 us).
        constexpr bool kAskGridInside = MODE == MODE_WEIGHT && R >= 6;
        if (!kRowByRow && !lattice && (MODE == MODE_WEIGHT || mode_codes_resident(MODE)) && p.wbits == 8) {
            // only stored: the packing instruction rounds and clamps (see pack4)
            uint32_t q[R] = {};
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!computed(r)) continue;
                const f4 gr = weight_grid(r);
                const MinMaxGrid grid = {gr[0], gr[2], gr[1]};
                float at[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) at[i] = weight_position_minmax(w[r][i], grid, xi);
                q[r] = pack4<8>(at);
            }
            store_packed(q, 8);
            continue;
        }
        if (!kAskGridInside && lattice) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (computed(r)) onto_lattice(r);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!computed(r)) continue;
                if (kAskGridInside && lattice) onto_lattice(r);
                else onto_minmax(r);
            }
        }
        if (emit) store_words(code, p.wbits);
        if (kWritesX && !keep_master) store(p.x, w);
        if (want16) store_half(p.x16, p.x16_f16 != 0u, w);
    }

    if (MODE != MODE_GRAD && !kLevels && args.n_saturated != nullptr) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) saturated += __shfl_down(saturated, off, 64);
        if ((threadIdx.x & 63) == 0 && saturated != 0) atomicAdd(args.n_saturated, (unsigned long long)saturated);
    }
}

}  // namespace qsdp
