// The learned-level encoders: a bucket is owned as in the wave kernels (qsdp_wave_kernel.hpp, whose loads, reductions
// and packing they share), its values are encoded against a table of K = 2^BITS ascending levels in [0, 1].
#pragma once

#include <type_traits>

#include "qsdp_wave_kernel.hpp"

namespace qsdp {

// Workgroups (of 4 waves) that a compute unit holds at once; the compiler has to leave room for them in registers.
constexpr int kLevelsResident = 5;

// ---------------------------------------------------------------------------------------
// Both encoders count bounds. The K-1 ascending BOUNDS of a table split the unit interval so that the number of bounds
// at or below a normalised value z is
//   * nearest level: the code. Bound k is the threshold between the levels k and k+1, the first value that is nearer to
//     the upper one, found exactly by trying the comparison of the two distances on the values next to the midpoint.
//   * coin flip: the lower enclosing level i. Bound k is the level k+1. A second LDS read fetches level i and the
//     reciprocal of its gap.
// Bounds, levels and values are in "cell units", scaled by the number of cells C, a power of two, so all comparisons,
// differences and products are the unscaled ones times an exact power of two and decide alike, bit for bit (but for
// normalised values below 2^-126, which the scaling saves from being rounded to subnormals).
//   * Counting by cell: for each of the C cells of the unit interval a table holds how many bounds lie at or below its
//     start and the next bound. If no cell holds two different bounds, a count is one LDS read and one comparison.
//     (Equal bounds, from equal levels, are passed all at once: the table also holds how many there are.)
//   * Counting by search, where a cell holds two: branch-free binary search whose first two pivots are
//     wave-uniform and held in scalar registers.
// Nearest-level tables whose thresholds cannot be relied on (see level_threshold) are searched by the plain definition.
// ---------------------------------------------------------------------------------------
enum LevelMethod { LEVELS_PLAIN = 0, LEVELS_BY_SEARCH = 1, LEVELS_BY_CELL = 2, LEVELS_BY_CELL_JUMPS = 3 };

template <int BITS>
struct LevelShape {
    static constexpr int K = 1 << BITS;
    // about eight cells to a bound: tables denser in the middle by a factor of four still have their cells to
    // themselves
    static constexpr int C = BITS <= 5 ? 256 : BITS == 6 ? 512 : 1024;
    static constexpr float kScale = (float)C;
};

struct LevelCell {
    float next;    // the first bound past the cell's start, +inf if none
    uint32_t count;  // bounds at or below the cell's start; upper half: bounds equal to `next`, less one
};

// What is wrong with a table, collected over the threads that set it up.
enum LevelFlags : uint32_t {
    LEVELS_UNUSABLE = 1u,  // a threshold that cannot be relied on
    LEVELS_CROWDED = 2u,   // a cell holds two different bounds
    LEVELS_JUMPS = 4u      // a cell holds equal bounds
};

// Entries thread, thread + THREADS, ... of the cell table over K - 1 bounds, K a power of two (cell c is [c, c+1) in
// cell units; the last entry, C, serves a value of exactly 1). All of a thread's entries are searched for side by
// side: the set-up is a chain of LDS reads, and small calls and small tensors wait for it.
template <int C, int THREADS>
__device__ __forceinline__ uint32_t fill_level_cells(LevelCell* cells, const float* bounds, int K, int thread) {
    constexpr int N = C / THREADS + 1;
    const int kb = K - 1;
    int at[N];  // ends as the number of bounds at or below the cell's start
#pragma unroll
    for (int i = 0; i < N; ++i) at[i] = 0;
    auto cell = [&](int i) { return thread + i * THREADS < C ? thread + i * THREADS : C; };
    for (int step = K >> 1; step >= 1; step >>= 1) {
        float bound[N];
#pragma unroll
        for (int i = 0; i < N; ++i) bound[i] = bounds[at[i] + step - 1];
#pragma unroll
        for (int i = 0; i < N; ++i) at[i] += bound[i] <= (float)cell(i) ? step : 0;
    }
    float next[N], after[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        next[i] = at[i] < kb ? bounds[at[i]] : __builtin_inff();
        after[i] = at[i] + 1 < kb ? bounds[at[i] + 1] : __builtin_inff();
    }
    uint32_t flags = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float end = (float)cell(i) + 1.0f;
        uint32_t equal = 0;  // bounds equal to `next`, less one, if that lies in the cell
        if (next[i] < end) {
            while (after[i] == next[i]) {
                ++equal;
                const int k = at[i] + 1 + (int)equal;
                after[i] = k < kb ? bounds[k] : __builtin_inff();
            }
            flags |= (after[i] < end ? LEVELS_CROWDED : 0u) | (equal != 0 ? LEVELS_JUMPS : 0u);
        }
        const LevelCell e = {next[i], (uint32_t)at[i] | (equal << 16)};
        cells[cell(i)] = e;
    }
    return flags;
}

// Threshold k of the K levels lv, scaled by `unit`; false if there is none to rely on. A value between the levels k
// and k+1 is compared with these two alone: one rounded distance rises with the value and the other falls, so the
// comparison flips once, and it does so within two steps of the midpoint (only the distance to a level below z/2 is
// rounded at all, by half a step). Values past the last level are compared with the last two: that goes to the last
// one if these are more than 2^-20 apart (the distances differ by the gap, and each is rounded by less than 2^-24),
// or equal, or if the last level is 1. In a run of equal levels every threshold is that of the run's end, so that its
// first level is the only one that is ever chosen.
__device__ __forceinline__ bool level_threshold(const float* lv, int k, int K, float unit, float* threshold) {
    const float lo = lv[k];
    int next = k + 1;
    while (next < K && lv[next] == lo) ++next;
    if (next == K) {
        *threshold = __builtin_inff();
        return lo >= 0.0f && lo <= unit;
    }
    const float hi = lv[next];
    auto upper = [&](float z) { return fabsf(z - hi) < fabsf(z - lo); };
    float t = 0.5f * (lo + hi);
    bool found = false;
    for (int i = 0; i < 8 && !found; ++i) {
        const float below = __uint_as_float(__float_as_uint(t) - 1u);
        if (!upper(t)) t = __uint_as_float(__float_as_uint(t) + 1u);
        else if (upper(below)) t = below;
        else found = true;
    }
    *threshold = t;
    const bool apart = hi - lo > 0x1p-20f * unit || hi == unit || lv[K - 1] != hi;
    return found && apart && lo >= 0.0f && hi <= unit;
}

// What the coin flip needs at level i: the level (cell units) and the reciprocal of the gap to the next one (per cell
// unit; 0 for the last level: nothing to round up to). The reciprocal is that of the unscaled gap, rounded (or
// infinite) as the definition has it, then divided by `cells`, exactly: (z - q) * rgap is the unscaled product bit
// for bit.
struct LevelCoin {
    float q, rgap;
};
__device__ __forceinline__ LevelCoin level_coin(const float* lv, int k, int K, float cells) {
    const float per_cell = 1.0f / cells;
    return {lv[k], k + 1 < K ? (1.0f / ((lv[k + 1] - lv[k]) * per_cell)) * per_cell : 0.0f};
}

// Whether the coin flip goes up: 2^16 - (h + 1/2) < 2^16 p for the 16-bit uniform h and p = (z - q) * rgap. Both
// sides are taken at 2^-16 of that, where the left one is exact and the right one cannot overflow for small gaps.
__device__ __forceinline__ bool coin_up(float z, float h, LevelCoin e) {
    return fmaf(h, -0x1p-16f, 1.0f - 0x1p-17f) < (z - e.q) * e.rgap;
}

// The bounds' first pivots. All lanes read the same addresses, so the values are wave-uniform and can live in SGPRs.
struct LevelPivots {
    float mid, lower, upper;
};
template <int BITS>
__device__ __forceinline__ LevelPivots load_level_pivots(const float* bounds) {
    constexpr int K = 1 << BITS;
    auto uniform = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
    return {uniform(bounds[K / 2 - 1]), uniform(bounds[BITS >= 2 ? K / 4 - 1 : 0]),
            uniform(bounds[BITS >= 2 ? 3 * K / 4 - 1 : 0])};
}

// How many bounds are at or below z (cell units). By cell the conversion saturates and the index is clamped, so a
// non-finite value cannot read outside the table.
template <int BITS, int METHOD>
__device__ __forceinline__ uint32_t count_bounds(float z, const float* bounds, const LevelCell* cells,
                                                 const LevelPivots& pv) {
    constexpr int K = 1 << BITS, C = LevelShape<BITS>::C;
    if constexpr (METHOD == LEVELS_BY_CELL || METHOD == LEVELS_BY_CELL_JUMPS) {
        const uint32_t c = (uint32_t)z;
        const LevelCell e = cells[c < (uint32_t)C ? c : (uint32_t)C];
        if constexpr (METHOD == LEVELS_BY_CELL) return e.count + (e.next <= z ? 1u : 0u);
        return (e.count & 0xFFFFu) + (e.next <= z ? (e.count >> 16) + 1u : 0u);
    } else {
        int j = pv.mid <= z ? K / 2 : 0;
        if (BITS >= 2) j += (j ? pv.upper : pv.lower) <= z ? K / 4 : 0;
#pragma unroll
        for (int step = K / 8; step >= 1; step >>= 1)
            if (bounds[j + step - 1] <= z) j += step;
        return (uint32_t)j;
    }
}

// A lane's rows: v -> codes.
template <int MODE, int G, int R, int BITS, int METHOD>
__device__ __forceinline__ void encode_levels_by(const float (&v)[R][4], uint32_t (&code)[R][4], float lo,
                                                 float inv_cells, const float* lv, const float* bounds,
                                                 const LevelCell* cells, const LevelCoin* coin,
                                                 const LevelPivots& pivots, uint64_t block_e0, int l, PhiloxKey key) {
    if constexpr (MODE == MODE_LEVELS_COIN) {
#pragma unroll
        for (int cp = 0; cp < R / 2; ++cp) {
            uint32_t h[4];
            grad_uniforms_rows<G, true>(block_e0, cp, l, key.k0, key.k1, h);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = 2 * cp + (i >> 2);
                const float z = (v[r][i & 3] - lo) * inv_cells;
                // Unbiased rounding onto the enclosing levels: with p = (z - level) / gap, up for the round(p * 2^16)
                // largest of the 2^16 values of the uniform h. z below the first level gives 0 (p < 0 there), at or
                // above the last K-1 (its reciprocal gap is 0).
                const uint32_t at = count_bounds<BITS, METHOD>(z, bounds, cells, pivots);
                const LevelCoin e = coin[at];
                code[r][i & 3] = at + (coin_up(z, (float)uniform16(h, i), e) ? 1u : 0u);
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = (v[r][i] - lo) * inv_cells;
                if constexpr (METHOD == LEVELS_PLAIN) code[r][i] = (uint32_t)nearest_level<BITS>(z, lv);
                else code[r][i] = count_bounds<BITS, METHOD>(z, bounds, cells, pivots);
            }
    }
}

// A workgroup takes a contiguous run of buckets (see level_blocks for how many), piece by piece of its tensors where
// every tensor has its own table (segs != nullptr), and its waves share the tables of the piece. What bounds the
// encoders: the instructions first, then the time a workgroup spends on its tables. Measured, 350M model in 292
// tensors (us; floor at 6.2 TB/s 265 / 258): 5 bit nearest 292, 4 bit coin flip 346, against 519 and 485 with tables
// of its own for every wave, set up for three buckets, and a second lookup (two levels and their distances) for the
// nearest level.
template <int MODE, int G, int R, int BITS, int W>
__global__ void __launch_bounds__(256, kLevelsResident) levels_kernel(const Params p,
                                                                       const Segment* __restrict__ segs) {
    static_assert(mode_is_levels(MODE), "mode");
    constexpr int T = 4 * G * R;  // elements of a bucket one wave holds
    constexpr int B = T * W;
    constexpr int BPW = 64 / G;
    constexpr int K = LevelShape<BITS>::K, C = LevelShape<BITS>::C;
    constexpr int kThreads = W == 1 ? 256 : 64 * W;  // the launch's workgroup size
    constexpr bool kCoin = MODE == MODE_LEVELS_COIN;
    constexpr int kTileBytes = 32 * R * BITS;
    __shared__ u4 stage_all[4 * kTileBytes / 16];
    __shared__ float red_all[W > 1 ? 2 * 2 * W : 1];  // [parity][lo/hi][wave]
    __shared__ float levels[K];
    __shared__ float thresholds[kCoin ? 1 : K];
    __shared__ LevelCoin coin[kCoin ? K : 1];
    __shared__ LevelCell cells[C + 1];
    __shared__ uint32_t table_flags;
    const float* bounds = kCoin ? levels + 1 : thresholds;
    const int lane = threadIdx.x & 63;
    const int sub = lane / G;
    const int l = lane % G;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* stage = reinterpret_cast<uint8_t*>(stage_all) + wave * kTileBytes;
    const uint32_t part0 = W > 1 ? wave * (uint32_t)T : 0u;
    const PhiloxKey key = launch_key<MODE>(p);
    const bool per_tensor = segs != nullptr;

    // the buckets of this workgroup; within a piece of them its waves (W > 1: the workgroup) take the units in turn
    uint64_t run = (p.num_buckets + gridDim.x - 1) / gridDim.x;
    if (run > BPW) run = (run + BPW - 1) / BPW * BPW;  // whole units, unless that would leave workgroups without work
    uint64_t begin = blockIdx.x * run;
    const uint64_t end = begin + run < p.num_buckets ? begin + run : p.num_buckets;
    const uint32_t q0 = W == 1 ? wave : 0u, q_step = W == 1 ? 4u : 1u;
    uint32_t tensor = 0;
    if (per_tensor && begin < end) find_segment(segs, p.nseg, begin, begin, &tensor);
    uint32_t parity = 0;
    while (begin < end) {
        Segment seg = {0, p.n, 0};
        uint64_t piece_end = end;
        if (per_tensor) {
            seg = segs[tensor];
            if (tensor + 1 < p.nseg && segs[tensor + 1].first_bucket < end) piece_end = segs[tensor + 1].first_bucket;
        }
        const uint64_t nunits = (piece_end - begin + BPW - 1) / BPW;
        struct UnitTile {
            bool active;      // the lane's bucket exists
            uint64_t bucket;  // the lane's bucket (the unit's first one for a lane without a bucket)
            uint64_t e0;      // first element of the wave's tile
            int m;            // elements of the tile that exist
            bool partial;     // wave-uniform: some lane's tile is short
        };
        auto unit_tile = [&](uint64_t q) -> UnitTile {
            UnitTile t;
            const uint64_t first = begin + q * BPW;
            t.active = first + sub < piece_end;
            t.bucket = t.active ? first + sub : first;
            const uint64_t local = (t.bucket - seg.first_bucket) * B;
            const uint64_t left = seg.n - local;
            const uint32_t m = left < (uint64_t)B ? (uint32_t)left : (uint32_t)B;
            t.e0 = seg.offset + local + part0;
            t.m = m > part0 ? (int)(m - part0 < (uint32_t)T ? m - part0 : (uint32_t)T) : 0;
            t.partial = __builtin_amdgcn_ballot_w64(t.m < T) != 0;
            return t;
        };
        // the values of the first unit are in flight while the tables are set up, those of the next one while a unit
        // is encoded
        float next[R][4];
        if (q0 < nunits) {
            const UnitTile t = unit_tile(q0);
            load_rows<G, R, false>(p.xin + t.e0, l, t.m, t.partial, next);
        }
        // tables of the piece
        const float* table = p.levels + (per_tensor ? (uint64_t)tensor * K : 0u);
        float mine[(K + kThreads - 1) / kThreads];
#pragma unroll
        for (int i = 0; i * kThreads < K; ++i) {
            const int k = threadIdx.x + i * kThreads;
            mine[i] = k < K ? table[k] : 0.0f;
        }
        __syncthreads();  // the tables of the piece before are no longer read
        if (threadIdx.x == 0) table_flags = 0;
#pragma unroll
        for (int i = 0; i * kThreads < K; ++i) {
            const int k = threadIdx.x + i * kThreads;
            if (k < K) levels[k] = mine[i] * LevelShape<BITS>::kScale;
        }
        __syncthreads();
        uint32_t found = 0;
        if constexpr (kCoin) {
            for (int k = threadIdx.x; k < K; k += kThreads)
                coin[k] = level_coin(levels, k, K, LevelShape<BITS>::kScale);
        } else {
            for (int k = threadIdx.x; k < K - 1; k += kThreads)
                if (!level_threshold(levels, k, K, LevelShape<BITS>::kScale, thresholds + k)) found |= LEVELS_UNUSABLE;
            __syncthreads();
        }
        found |= fill_level_cells<C, kThreads>(cells, bounds, K, threadIdx.x);
        if (found != 0) atomicOr(&table_flags, found);
        __syncthreads();
        const uint32_t flags = __builtin_amdgcn_readfirstlane(table_flags);
        const int method = flags & LEVELS_UNUSABLE ? LEVELS_PLAIN  // workgroup-uniform
                         : flags & LEVELS_CROWDED  ? LEVELS_BY_SEARCH
                         : flags & LEVELS_JUMPS    ? LEVELS_BY_CELL_JUMPS
                                                   : LEVELS_BY_CELL;
        const LevelPivots pivots = load_level_pivots<BITS>(bounds);

        for (uint64_t q = q0; q < nunits; q += q_step, parity ^= 1u) {
            const UnitTile tile = unit_tile(q);
            const uint64_t first = begin + q * BPW;
            const int active_buckets = piece_end - first < (uint64_t)BPW ? (int)(piece_end - first) : BPW;
            const uint64_t tile_slot0 = (W == 1 ? first : tile.bucket) * (uint64_t)B + part0;
            u4* tile_out = reinterpret_cast<u4*>(reinterpret_cast<uint8_t*>(p.codes) + (tile_slot0 >> 3) * BITS);
            float v[R][4];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[r][i] = next[r][i];
            if (q + q_step < nunits) {
                const UnitTile t = unit_tile(q + q_step);
                load_rows<G, R, false>(p.xin + t.e0, l, t.m, t.partial, next);
            }
            float lo, hi;
            rows_minmax<G, R, false>(v, l, tile.m, tile.partial, lo, hi);
            block_combine_minmax<W>(lo, hi, red_all + (W > 1 ? parity * 2 * W : 0), wave);
            const MinMaxGrid grid = make_minmax_grid(lo, hi, 1.0f, false);  // scale = hi - lo, inv = 1/(hi - lo)
            // normalised value in cell units: (v - lo) * inv_cells
            const float inv_cells = grid.inv * LevelShape<BITS>::kScale;
            const uint64_t block_e0 = p.block0 + (tile.e0 >> 3);  // Philox block of the tile's first element
            uint32_t code[R][4];
            // the method is chosen once for all of the lane's elements, so that each is straight-line code over the
            // rows and the LDS reads of different elements overlap
            auto encode = [&](auto by) {
                encode_levels_by<MODE, G, R, BITS, decltype(by)::value>(v, code, grid.lo, inv_cells, levels, bounds,
                                                                        cells, coin, pivots, block_e0, l, key);
            };
            if (__builtin_expect(method == LEVELS_BY_CELL, 1)) encode(std::integral_constant<int, LEVELS_BY_CELL>{});
            else if (method == LEVELS_BY_CELL_JUMPS) encode(std::integral_constant<int, LEVELS_BY_CELL_JUMPS>{});
            else if (kCoin || method == LEVELS_BY_SEARCH) encode(std::integral_constant<int, LEVELS_BY_SEARCH>{});
            else encode(std::integral_constant<int, LEVELS_PLAIN>{});
            if (__builtin_expect(tile.partial, 0)) zero_slots_past_end<G, R, false>(code, l, tile.m);
            store_codes<G, R, BITS>(stage, tile_out, lane, active_buckets, code);
            if (tile.active && l == 0 && (W == 1 || wave == 0)) {
                p.meta[2 * tile.bucket] = grid.lo;
                p.meta[2 * tile.bucket + 1] = grid.scale;
            }
        }
        begin = piece_end;
        ++tensor;
    }
}

}  // namespace qsdp
