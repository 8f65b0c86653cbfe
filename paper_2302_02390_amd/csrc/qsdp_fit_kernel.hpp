// Level fitting (Algorithm 1 in batched form).
#pragma once

#include "qsdp_params.hpp"

namespace qsdp {

// ---------------------------------------------------------------------------------------
// Level fitting: a workgroup walks the buckets of its tensor in order, since every batch starts from the levels the
// previous one left. Per batch every value goes to its nearest level (levels frozen); level k then takes its count_k
// steps of rate lr towards the mean of its values at once, in binary64: q <- q - (1 - (1-lr)^c)(q - mean), with the
// mean of exact 32.32 fixed-point sums.
//
// The serial chain of batches bounds this, so the chain holds as little as possible. What a batch needs from the
// levels is, for each pair of neighbours, how many values lie on the lower one's side and their sum; the normalised
// values themselves do not depend on the levels. Producer waves therefore sort the coming batches into cells of the
// unit interval (a counting sort: one LDS atomic per value returns the place within the cell and adds up count and
// sum, packed into one word; a prefix sum over the cells follows), and one consumer wave walks the chain: a lane per
// pair of neighbours reads the prefix at the cell of the midpoint, compares the few values of that cell with the two
// levels, and has count and sum below the boundary; differences between lanes are the levels' own. No barrier and no
// atomic is left in the chain; two LDS round trips for the boundary, one for the powers of 1 - lr and the reciprocals
// of the counts. A team of W producer waves sorts a batch (the values stay in registers, at most 16 to a lane) and P
// teams make a round: W = 1, P = 6 or 7 for buckets of up to 1024 values (one wave needs no barrier between its passes;
// at 1024 six sort more slowly than the consumer walks: 0.53 us per batch, 5 bits, where seven take 0.48, and eight are
// no faster), W = 2, 4, 8 and P = 8 / W up to 2048, 4096, 8192 with a barrier after each of the four passes. The
// consumer meanwhile walks the P batches of the round before; the slots are double-buffered.
//
// Measured (us per batch, 5-bit table, Gaussian values, buckets of 128 / 352 / 1024 / 4096 / 8192): 0.40 / 0.43 / 0.48
// / 1.73 / 3.3, against 1.27 / - / 2.6 / 10.7 / 21 for a workgroup that stages one batch in LDS and assigns value by
// value with a barrier around each part; the 292 tables of the 350M model 2.85 -> 0.51 ms. The chain is latency: about
// 950 cycles of dependent LDS reads, comparisons and binary64 steps per batch. Beyond 512 values the sorting binds,
// with LDS in use for half of the cycles (1024 / 4096: 607 of 1,170, 2,090 of 4,160, bank conflicts 340 and 1,240 of
// them; an atomic, a read and a write to random places take 15 + 16 + 11 cycles for the 64 lanes of a wave) and
// producers that wait for their answers pass after pass in the rest. Lanes without a value make no access: on one
// place, as they did when they added zero to their neighbour's cell, they meet in turn (buckets of 352 / 736, 5 bit:
// 0.56 / 0.69 -> 0.43 / 0.50 us per batch, 3040, 4 bit: 2.4 -> 1.8).
// Tensors of few batches are bound by what a workgroup does before its first one, the table of powers above all (one
// batch of 1024, 4 bit: 32 us when the whole table was filled first, 10 us now, against 16 us for the workgroup that
// staged its batches), and by one workgroup of this size to a compute unit: 2000 such tensors 240 -> 46 us (53 us then;
// 2 bit, whose counts ask for more powers: 240 -> 103 us, 57 us then). Producers without a batch sort nothing (they
// sorted the last one again: 2000 tensors of one batch of 512, 4 bit, 25.8 -> 20.2 us).
//
// The boundary search needs levels that ascend by more than 2^-20 within [0, 1] (then the comparison of the two
// rounded distances is monotone in the value and flips within 2^-22 of the midpoint) and cells that are not
// crowded. A batch for which that does not hold is assigned value by value, by the same wave.
// ---------------------------------------------------------------------------------------
struct FitParams {
    const float* v;
    float* levels;  // in/out, 2^bits floats (one table per tensor when segs is given)
    uint64_t n;
    uint64_t num_batches;  // with segs: the cap on the batches of every tensor (0 = none)
    const Segment* segs;   // multi-tensor fit: workgroup t fits tensor t on its own table
    int bucket;
    int bits;
    float lr;
};

// Shape of a workgroup: W waves to a batch of up to 64 * W * VPT values.
template <int BMAX, int C>
struct FitSlot;

template <int BITS, int VPT, int W>
struct FitShape {
    static constexpr int kBucketMax = 64 * W * VPT;
    // Buckets of 129-256 keep six producers: seven ask for more than a third of a compute unit's LDS, and the chain is
    // no faster with them (us, six / seven, 5 bits, buckets of 160 and 256: 400 batches of one tensor 163 / 163, 164 /
    // 163, 700 tensors of two 8.6 / 11.5, 8.7 / 11.6; 2000 of three at 8 bits 30 / 37, 32 / 40). So do tables of up to
    // 8 levels with buckets of 257-512: 200 tensors of one bucket of 512, 1 / 2 / 3 bits, 9.6 / 11.8, 8.3 / 10.0, 6.5
    // / 7.3, 400 batches of one tensor 173 / 173, 178 / 180, 177 / 178 (at 4 bits seven are faster: 2000 tensors 17.1
    // for 18.8).
    static constexpr bool kSixProducers = VPT == 4 || (VPT == 8 && BITS <= 3);
    static constexpr int kBatches = W > 1 ? 8 / W : kSixProducers ? 6 : 7;  // P, batches per round
    static constexpr int kProducers = kBatches * W;              // producer waves; the consumer is one more
    static constexpr int kThreads = 64 * (kProducers + 1);
    static constexpr int kBarriers = W == 1 ? 1 : 4;             // per round
    // About a cell per value, as far as the 2 P slots leave LDS to spare. Half of that for buckets of 512 and up to
    // 16 levels, where it lets two workgroups share a compute unit at no cost to the chain (2000 tensors of one
    // batch, 4 bit: 33.7 -> 23.3 us; with more levels the chain loses: 5 bit 0.49 -> 0.53 us per batch, 6 bit 0.56 ->
    // 0.65).
    static constexpr int kCells = kBucketMax <= 256                ? kBucketMax
                                  : kBucketMax == 512 && BITS <= 4 ? 256
                                  : kBucketMax <= 2048             ? 512
                                                                   : 1024;
    using Slot = FitSlot<kBucketMax, kCells>;
};

// Count and sum of a set of normalised values in one word: sum of at most 2^13 values of at most 2^32 below, count
// above.
constexpr int kFitCountShift = 46;
constexpr uint64_t kFitSumMask = (1ull << kFitCountShift) - 1;

// What follows the values of a batch: above every boundary, as many as the consumer reads at once.
constexpr float kFitFiller = 2.0f;
constexpr int kFitSpare = 16;

// z (in [0, 1]) in 32.32 fixed point, truncated: exact scaling, the integer and the fraction converted apart.
__device__ __forceinline__ uint64_t fit_fixed(float z) {
    const uint32_t whole = (uint32_t)z;
    return ((uint64_t)whole << 32) | (uint32_t)((z - (float)whole) * 4294967296.0f);
}

// The cell of a value (or of a boundary): C cells of equal width from `from` on, what lies outside them in the first
// and the last. Monotone, and in range whatever the argument (the conversion saturates).
struct FitCells {
    float from, per_unit;
};
template <int C>
__device__ __forceinline__ uint32_t fit_cell(float z, FitCells cells) {
    const uint32_t c = (uint32_t)((z - cells.from) * cells.per_unit);
    return c < (uint32_t)C ? c : (uint32_t)(C - 1);
}

// The cells for a batch: over its mean +- four times its mean magnitude, within its range [lo, hi]. That is the whole
// range for Gaussian weights; for heavy-tailed gradients it keeps the cells where the values are (a range stretched
// by one outlier would put most of a batch into a few cells).
template <int C>
__device__ __forceinline__ FitCells fit_cells(const MinMaxGrid& grid, float hi, float mean, float magnitude) {
    const float from = fmaxf(grid.lo, mean - 4.0f * magnitude);
    const float to = fminf(hi, mean + 4.0f * magnitude);
    const float width = (to - from) * grid.inv;
    const FitCells inner = {(from - grid.lo) * grid.inv, (float)C / width};
    const FitCells all = {0.0f, (float)C};
    return width > 0x1p-20f && width <= 2.0f ? inner : all;
}

// v of the next / previous lane of the wave (the last / first lane gets 0).
__device__ __forceinline__ uint32_t next_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, true);  // wave_shl:1
}
__device__ __forceinline__ uint32_t previous_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);  // wave_shr:1
}

// Sum over the lanes of a wave, in all of them (any order: it only places the cells).
__device__ __forceinline__ float fit_wave_sum(float v) {
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    float a, b;
    swap16(v, a, b);
    v = a + b;
    swap32(v, a, b);
    return a + b;
}

// Inclusive prefix sum over the lanes of a wave.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t fit_scan_step(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xF, false);
    return v + (((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ uint64_t fit_wave_scan(uint64_t v) {
    v = fit_scan_step<0x111, 0xF>(v);  // row_shr:1, 2, 4, 8: within rows of 16 lanes
    v = fit_scan_step<0x112, 0xF>(v);
    v = fit_scan_step<0x114, 0xF>(v);
    v = fit_scan_step<0x118, 0xF>(v);
    v = fit_scan_step<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v = fit_scan_step<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Sum over the lanes l, l + 64/S, l + 2 * 64/S, ... (S = 1, 2, 4).
template <int S>
__device__ __forceinline__ uint64_t fit_sum_subs(uint64_t v) {
    if constexpr (S >= 2) {
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
        v = (((uint64_t)hi[0] << 32) | lo[0]) + (((uint64_t)hi[1] << 32) | lo[1]);
    }
    if constexpr (S >= 4) {
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
        v = (((uint64_t)hi[0] << 32) | lo[0]) + (((uint64_t)hi[1] << 32) | lo[1]);
    }
    return v;
}

// Adds to a word in LDS and returns what it held. Relaxed: the callers put their own fences, and an ordered atomic
// would wait for each one before the next.
__device__ __forceinline__ uint64_t fit_add(uint64_t* word, uint64_t v) {
    return __hip_atomic_fetch_add(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// LDS traffic of one wave is processed in order; this keeps the compiler from reordering it.
__device__ __forceinline__ void fit_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (1 - lr)^c by repeated multiplication, the order in which c single steps compound, for c up to the bucket size:
// every power up to kFine beside the reciprocal of the count, beyond that every kStep-th. The multiplications are a
// serial chain (about 8 ns each), so the consumer extends it as the counts ask for it: most counts are a small share
// of a bucket, and a tensor of few batches would wait for powers that it never reads. The reciprocals are the
// producers' work, while their first loads are on the way.
struct FitFilled {
    int count;    // the powers of counts up to this one can be read
    double keep;  // where the chain stands
};
template <int BMAX>
struct FitPowers {
    static constexpr int kFine = BMAX < 1024 ? BMAX : 1024, kStep = 16, kCoarse = (BMAX - kFine) / kStep + 1;
    static_assert(kFine % 64 == 0, "grows by 64");
    struct Entry {
        double moved, reciprocal;  // 1 - (1-lr)^c, 1 / c
    };
    Entry fine[kFine + 1];
    double coarse[kCoarse];

    __device__ void fill_reciprocals(int top, int thread, int threads) {
        for (int c = thread; c <= kFine && c <= top; c += threads) fine[c].reciprocal = 1.0 / (double)(c > 0 ? c : 1);
    }

    __device__ FitFilled start(int lane) {
        if (lane == 0) fine[0].moved = 0.0;
        return {0, 1.0};
    }

    // The next 64 powers, or the next 16 of every kStep-th (one wave; the chain and its stores in one lane).
    __device__ void extend(FitFilled& f, double one_minus, int lane) {
        double keep = f.keep;
        if (f.count < kFine) {
            if (lane == 0) {
                uint32_t first = (uint32_t)f.count + 1u;
                asm volatile("" : "+v"(first));  // one address register, the stores' offsets in the instructions
#pragma unroll 16
                for (int i = 0; i < 64; ++i) {
                    keep *= one_minus;
                    fine[first + i].moved = keep;
                }
            }
            fit_wave_sync();
            double& mine = fine[f.count + 1 + lane].moved;
            mine = 1.0 - mine;
            f.count += 64;
        } else {
            const int first = (f.count + 1 - kFine) / kStep;
            if (lane == 0) {
                for (int k = first; k < first + 16; ++k) {
                    if (k < kCoarse) coarse[k] = keep;
#pragma unroll
                    for (int i = 0; i < kStep; ++i) keep *= one_minus;
                }
            }
            f.count = kFine + (first + 16) * kStep - 1;
        }
        const uint64_t bits = __builtin_bit_cast(uint64_t, keep);
        const uint64_t low = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)bits);
        const uint64_t high = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(bits >> 32));
        f.keep = __builtin_bit_cast(double, (high << 32) | low);
        fit_wave_sync();
    }

    // Where the level q lands after the c values of fixed-point sum `total` that are its own; c at most kFine. Without
    // values it stays, whatever it holds.
    static __device__ __forceinline__ float step(float level, uint32_t c, uint64_t total, Entry e) {
        // total / c rounded once: t * (1/c) is off by at most 2 ulp, the remainder is exact (c is below 2^11, so it has
        // at most 12 bits more than an ulp), and the corrected quotient is within 2^-50 ulp of t / c, which, t and c
        // being integers below 2^46 and 2^11, is never closer than 2^-12 ulp to a rounding boundary without being
        // a binary64 number itself
        const double q = (double)level, t = (double)total;
        const double a = t * e.reciprocal;
        const double mean = fma(fma(-a, (double)c, t), e.reciprocal, a) * (1.0 / 4294967296.0);
        return c == 0u ? level : (float)(q - e.moved * (q - mean));
    }

    // The same for any c.
    __device__ float step_any(float level, uint32_t c, uint64_t total, double one_minus) const {
        if (c <= (uint32_t)kFine) return step(level, c, total, fine[c]);
        const int k = ((int)c - kFine) / kStep;
        double keep = coarse[k];
        for (int i = kFine + k * kStep; i < (int)c; ++i) keep *= one_minus;
        const double q = (double)level;
        const double mean = ((double)total / (double)c) * (1.0 / 4294967296.0);
        return c == 0u ? level : (float)(q - (1.0 - keep) * (q - mean));
    }
};

// A batch as the consumer reads it: the values grouped by cell (ascending cells, any order within one), and for every
// cell count and sum of the values in the cells before it; cell C: of all values.
// The prefix sum gives a lane kOwn cells in a row; one word of padding after each of these runs keeps the lanes off
// one another's banks (without it all 64 lanes meet in two banks: 0.15 us more per batch of 1024).
template <int BMAX, int C>
struct FitSlot {
    static constexpr int kValues = BMAX;
    static constexpr int kOwn = C / 64;
    static __device__ __forceinline__ uint32_t at(uint32_t c) { return c + (kOwn > 1 ? c / kOwn : 0u); }
    uint64_t cell[C + 64 + 1];  // cell c at at(c)
    float z[BMAX + kFitSpare];  // grouped by cell, kFitSpare fillers past the last one
    FitCells cells;
};

// Level k of the table for lane l: k = 64 * i + (l mod (64 / S)), i < M. S lanes share a level's work.
template <int BITS>
struct FitLanes {
    static constexpr int K = 1 << BITS;
    static constexpr int S = K <= 16 ? 4 : K <= 32 ? 2 : 1;
    static constexpr int M = K <= 64 ? 1 : K / 64;
};

// One batch of the chain. lv[i]: the lane's levels, updated. lv_shared, acc: K entries of LDS each, for batches that
// are assigned value by value.
template <int BITS, typename Slot, typename Powers, int C>
__device__ __forceinline__ void fit_batch(const Slot& slot, int m, Powers& powers, FitFilled& filled, double one_minus,
                                          FitCells cells, float (&lv)[FitLanes<BITS>::M], float* lv_shared,
                                          uint64_t* acc, int lane) {
    constexpr int K = FitLanes<BITS>::K, S = FitLanes<BITS>::S, M = FitLanes<BITS>::M;
    // Values a lane reads at once, one after the other in the slot: one address, no question of range (below), half
    // the instructions of a read, test and sum for each on its own (6 bits 0.66 -> 0.59 us per batch of 1024, 5 bits
    // 0.43 -> 0.40 per batch of 128). Eight of them where two lanes share a level are slower (0.46).
    constexpr int U = M == 4 ? 2 : 4;
    static_assert(S * U <= kFitSpare, "reads past the last value");
    // values in a boundary's cells from which the plain assignment of the batch is faster
    const uint32_t crowded = (uint32_t)(m * S * U / (48 * M)) + 64u;
    const int sub = S > 1 ? lane / (64 / S) : 0;
    const int k0 = S > 1 ? lane % (64 / S) : lane;
    uint64_t upto[M];  // count and sum of the values of levels 0 .. k
    float hi[M];
    uint32_t pos[M], end[M];
    bool plain = false;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const int k = 64 * i + k0;
        hi[i] = __uint_as_float(next_lane(__float_as_uint(lv[i])));
        if (i + 1 < M) {
            const float following = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lv[i + 1 < M ? i + 1 : 0]), 0));
            hi[i] = lane == 63 ? following : hi[i];
        }
        const bool inner = k < K - 1;
        const bool ok = inner ? hi[i] - lv[i] > 0x1p-20f && lv[i] >= 0.0f && hi[i] <= 1.0f : true;
        const float mid = 0.5f * (lv[i] + hi[i]);
        // past the last boundary: everything, no value left to compare
        const uint32_t first = inner ? fit_cell<C>(mid - 0x1p-21f, cells) : (uint32_t)C;
        const uint32_t last = inner ? fit_cell<C>(mid + 0x1p-21f, cells) + 1u : (uint32_t)C;
        upto[i] = slot.cell[Slot::at(first)];
        end[i] = (uint32_t)(slot.cell[Slot::at(last)] >> kFitCountShift);
        pos[i] = (uint32_t)(upto[i] >> kFitCountShift);
        plain = plain || !ok || end[i] - pos[i] > crowded;
    }
    uint64_t own[M];
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(plain) == 0, 1)) {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            // The values at `end` and beyond are those of higher cells, or the fillers past the last one: above the
            // boundary, so they may be read with the others. A lane past the last boundary compares with levels that
            // have nothing on the lower one's side.
            const bool inner = 64 * i + k0 < K - 1;
            const float below_level = inner ? lv[i] : -4.0f, above_level = inner ? hi[i] : kFitFiller;
            uint64_t below = 0;
            uint32_t p = pos[i];
            do {
                const float* at = &slot.z[p + sub * U];
                float z[U];
#pragma unroll
                for (int u = 0; u < U; ++u) z[u] = at[u];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    // on the lower level's side: below 1 (the upper level is at most 1 and closer), so 32 bits hold it
                    const bool lower = !(fabsf(z[u] - above_level) < fabsf(z[u] - below_level));
                    const uint32_t fixed = (uint32_t)(z[u] * 4294967296.0f);
                    below += ((uint64_t)(lower ? 1u << (kFitCountShift - 32) : 0u) << 32) | (lower ? fixed : 0u);
                }
                p = p + S * U < end[i] ? p + S * U : end[i];  // the lanes that are done: nothing below any more
            } while (__builtin_amdgcn_ballot_w64(p < end[i]) != 0);
            upto[i] += fit_sum_subs<S>(below);
        }
#pragma unroll
        for (int i = 0; i < M; ++i) {
            uint32_t lo_prev = previous_lane((uint32_t)upto[i]), hi_prev = previous_lane((uint32_t)(upto[i] >> 32));
            if (i > 0) {
                const uint64_t preceding = upto[i > 0 ? i - 1 : 0];
                const uint32_t lo_63 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)preceding, 63);
                const uint32_t hi_63 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(preceding >> 32), 63);
                lo_prev = lane == 0 ? lo_63 : lo_prev;
                hi_prev = lane == 0 ? hi_63 : hi_prev;
            }
            const uint64_t prev = 64 * i + k0 == 0 ? 0ull : ((uint64_t)hi_prev << 32) | lo_prev;
            own[i] = upto[i] - prev;
        }
    } else {
        // value by value against the table in LDS
        fit_wave_sync();
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = 64 * i + k0;
            if (sub == 0 && k < K) {
                lv_shared[k] = lv[i];
                acc[k] = 0;
            }
        }
        fit_wave_sync();
        for (int p = lane; p < m; p += 64 * 4) {  // four values a lane at once: the searches' LDS reads overlap
            float z[4];
            int k[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) z[u] = slot.z[p + 64 * u < m ? p + 64 * u : p];
#pragma unroll
            for (int u = 0; u < 4; ++u) k[u] = nearest_level<BITS>(z[u], lv_shared);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (p + 64 * u < m) fit_add(&acc[k[u]], (1ull << kFitCountShift) | fit_fixed(z[u]));
        }
        fit_wave_sync();
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = 64 * i + k0;
            own[i] = k < K ? acc[k] : 0;
        }
        fit_wave_sync();
    }
    // the powers are requested before it is known whether the table holds them: the answer comes while they are on
    // the way
    uint32_t c[M], most = 0;
    typename Powers::Entry e[M];
    auto request = [&] {
#pragma unroll
        for (int i = 0; i < M; ++i) e[i] = powers.fine[c[i] < (uint32_t)Powers::kFine ? c[i] : (uint32_t)Powers::kFine];
    };
#pragma unroll
    for (int i = 0; i < M; ++i) {
        c[i] = (uint32_t)(own[i] >> kFitCountShift);
        most = c[i] > most ? c[i] : most;
    }
    request();
    if (filled.count < m) {
        while (__builtin_expect(__builtin_amdgcn_ballot_w64(most > (uint32_t)filled.count) != 0, 0)) {
            powers.extend(filled, one_minus, lane);
            request();
        }
    }
    if (Powers::kFine == Slot::kValues ||
        __builtin_expect(__builtin_amdgcn_ballot_w64(most > (uint32_t)Powers::kFine) == 0, 1)) {
#pragma unroll
        for (int i = 0; i < M; ++i) lv[i] = Powers::step(lv[i], c[i], own[i] & kFitSumMask, e[i]);
    } else {
#pragma unroll
        for (int i = 0; i < M; ++i) lv[i] = powers.step_any(lv[i], c[i], own[i] & kFitSumMask, one_minus);
    }
}

template <int BITS, int VPT, int W>
__global__ void __launch_bounds__((FitShape<BITS, VPT, W>::kThreads)) fit_levels_kernel(const FitParams p) {
    using Shape = FitShape<BITS, VPT, W>;
    using Slot = typename Shape::Slot;
    constexpr int C = Shape::kCells, P = Shape::kBatches, K = 1 << BITS;
    constexpr int M = FitLanes<BITS>::M, S = FitLanes<BITS>::S;
    __shared__ Slot slots[2 * P];
    typedef FitPowers<Shape::kBucketMax> Powers;
    __shared__ Powers powers;
    __shared__ float lv_shared[K];
    __shared__ uint64_t acc[K];
    __shared__ float red[P][4][W];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int B = p.bucket;
    // this workgroup's tensor: the whole vector, or tensor blockIdx.x of a multi-tensor fit
    const float* v = p.v;
    float* levels = p.levels;
    uint64_t n = p.n, num_batches = p.num_batches;
    if (p.segs != nullptr) {
        const Segment seg = p.segs[blockIdx.x];
        v += seg.offset;
        levels += (uint64_t)blockIdx.x * K;
        n = seg.n;
        num_batches = (n + (uint64_t)B - 1) / (uint64_t)B;
        if (p.num_batches > 0 && p.num_batches < num_batches) num_batches = p.num_batches;
    }
    if (num_batches == 0) return;
    auto batch_size = [&](uint64_t j) -> int {  // j < num_batches
        const uint64_t left = n - j * (uint64_t)B;
        return left < (uint64_t)B ? (int)left : B;
    };
    const uint64_t rounds = (num_batches + P - 1) / P;  // of the consumer; the producers are one ahead
    const double one_minus = 1.0 - (double)p.lr;

    if (wave == Shape::kProducers) {
        // the consumer: round r walks the batches that were sorted in round r - 1
        __builtin_amdgcn_s_setprio(3);
        float lv[M];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = 64 * i + (S > 1 ? lane % (64 / S) : lane);
            lv[i] = k < K ? levels[k] : 0.0f;
        }
        FitFilled filled = powers.start(lane);
        // while the producers sort the first round: up to three times the mean count, which the fullest level of a
        // Gaussian batch on the uniform table does not reach; all of them for the smallest buckets
        while (filled.count < Powers::kFine && (Powers::kFine <= 256 || filled.count * K < 3 * B))
            powers.extend(filled, one_minus, lane);
        for (int i = 0; i < Shape::kBarriers; ++i) __syncthreads();  // the producers' first round
        for (uint64_t r = 0; r < rounds; ++r) {
            const int buffer = (int)(r & 1u) * P;
            FitCells cells[P];
#pragma unroll
            for (int i = 0; i < P; ++i) cells[i] = slots[buffer + i].cells;
#pragma unroll
            for (int i = 0; i < P; ++i) {
                if (r * P + i < num_batches)
                    fit_batch<BITS, Slot, Powers, C>(slots[buffer + i], batch_size(r * P + i), powers, filled,
                                                     one_minus, cells[i], lv, lv_shared, acc, lane);
                for (int b = 0; b < (W == 1 ? (i == P - 1 ? 1 : 0) : Shape::kBarriers / P); ++b) __syncthreads();
            }
        }
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = 64 * i + (S > 1 ? lane % (64 / S) : lane);
            if ((S == 1 || lane < 64 / S) && k < K) levels[k] = lv[i];
        }
    } else {
        // between the passes of a team
        auto team_sync = [] {
            if constexpr (W > 1) __syncthreads(); else fit_wave_sync();
        };
        // a producer: batch r * P + team in round r, this wave's 1/W of it; nothing but the barriers past the last one.
        // Lanes past the end of a batch fetch its last value, which changes no minimum or maximum, and enter nothing.
        const int team = wave / W, part = wave % W;
        const int scanner = W == 2 ? team / 2 : W == 4 ? team : 0;  // of the team's waves: on another SIMD for every team
        const int first = part * 64 + lane;  // value q of the lane: first + q * 64 * W
        float next[VPT];
        auto batch = [&](uint64_t r) -> uint64_t { return r * P + team; };
        auto fetch = [&](uint64_t j) {
            const int m = batch_size(j);
            const float* src = v + j * (uint64_t)B;
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                const int i = first + q * 64 * W;
                next[q] = src[i < m ? i : m - 1];
            }
        };
        fetch(batch(0) < num_batches ? batch(0) : num_batches - 1);
        powers.fill_reciprocals(B, threadIdx.x, 64 * Shape::kProducers);
        for (uint64_t r = 0; r <= rounds; ++r) {
            if (batch(r) >= num_batches) {  // the consumer's last round among them
                for (int i = 0; i < Shape::kBarriers; ++i) __syncthreads();
                continue;
            }
            const int m = batch_size(batch(r));
            Slot& slot = slots[(int)(r & 1u) * P + team];
            float z[VPT];
            float lo = next[0], hi = next[0], sum = 0.0f, absolute = 0.0f;
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                z[q] = next[q];
                lo = fminf(lo, z[q]);
                hi = fmaxf(hi, z[q]);
                sum += z[q];
                absolute += fabsf(z[q]);
            }
            fetch(batch(r + 1) < num_batches ? batch(r + 1) : num_batches - 1);  // in flight while this batch is sorted
            for (int c = first; c < C + 64; c += 64 * W) slot.cell[c] = 0;  // all but the last, written below
            lo = group_min<64>(lo);
            hi = group_max<64>(hi);
            sum = fit_wave_sum(sum);
            absolute = fit_wave_sum(absolute);
            if constexpr (W > 1) {
                if (lane == 0) {
                    red[team][0][part] = lo;
                    red[team][1][part] = hi;
                    red[team][2][part] = sum;
                    red[team][3][part] = absolute;
                }
                __syncthreads();
                sum = absolute = 0.0f;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    lo = fminf(lo, red[team][0][w]);
                    hi = fmaxf(hi, red[team][1][w]);
                    sum += red[team][2][w];
                    absolute += red[team][3][w];
                }
            } else {
                fit_wave_sync();
            }
            const MinMaxGrid grid = make_minmax_grid(lo, hi, 1.0f, false);
            const FitCells cells = fit_cells<C>(grid, hi, sum * (1.0f / (64 * W * VPT)), absolute * (1.0f / (64 * W * VPT)));
            uint32_t cell[VPT];
            uint64_t held[VPT];  // the cell's word before this value came (both halves used: half of one dropped costs a wait)
            auto enter = [&](int q) {
                z[q] = (z[q] - grid.lo) * grid.inv;
                cell[q] = Slot::at(fit_cell<C>(z[q], cells));
                held[q] = fit_add(&slot.cell[cell[q]], (1ull << kFitCountShift) | fit_fixed(z[q]));
            };
            const bool full = m == Shape::kBucketMax;
            if (full) {
#pragma unroll
                for (int q = 0; q < VPT; ++q) enter(q);
            } else {
#pragma unroll
                for (int q = 0; q < VPT; ++q)
                    if (first + q * 64 * W < m) enter(q);
            }
            team_sync();
            if (part == scanner) {
                constexpr int kOwn = Slot::kOwn;
                uint64_t* own = &slot.cell[Slot::at(lane * kOwn)];
                uint64_t before[kOwn], total = 0;
#pragma unroll
                for (int c = 0; c < kOwn; ++c) {
                    before[c] = total;
                    total += own[c];
                }
                const uint64_t incl = fit_wave_scan(total);
#pragma unroll
                for (int c = 0; c < kOwn; ++c) own[c] = before[c] + (incl - total);
                if (lane == 63) slot.cell[Slot::at(C)] = incl;
                if (lane == 0) slot.cells = cells;
            }
            team_sync();
            auto place = [&](int q) {
                slot.z[(uint32_t)((slot.cell[cell[q]] + held[q]) >> kFitCountShift)] = z[q];
            };
            if (full) {
#pragma unroll
                for (int q = 0; q < VPT; ++q) place(q);
            } else {
#pragma unroll
                for (int q = 0; q < VPT; ++q)
                    if (first + q * 64 * W < m) place(q);
            }
            if (part == 0 && lane < kFitSpare) slot.z[m + lane] = kFitFiller;
            __syncthreads();
        }
    }
}

}  // namespace qsdp
