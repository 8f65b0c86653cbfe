// Level fitting (Algorithm 1 in batched form).
#pragma once

#include <type_traits>

#include "qsdp_fit_common.hpp"

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
// unit interval (a counting sort: one LDS atomic per value returns the place within the cell, a prefix sum over the
// cells follows), with count and sum before every fourth value of the sorted batch, and one consumer wave walks the
// chain: a lane per pair of neighbours reads where the cell of the midpoint starts, compares the few values from there
// on with the boundary, and adds what lies before them; differences between lanes are the levels' own.
//
// A producer sorts a batch of up to 2048 values by itself (up to 32 to a lane, in registers; larger buckets:
// qsdp_fit_rounds.hpp), so its passes need no barrier. P producers and the consumer share a ring of slots: a producer
// starts on a slot when the consumer has counted the batch that it held as read, the consumer on a batch when the slot
// shows its number. Both words are in LDS, whose accesses are processed in order for each wave, and all waves of the
// workgroup are resident, so every wait ends. With a barrier per round of P batches in its place, and slots for two
// rounds, the consumer waited for the slowest producer of each round.
//
// What bounds the chain is latency, in this order: an instruction that needs the result of the one before waits 8
// cycles for it (others issue every 4), an LDS read takes 56-70, a branch on a lane's comparison 36, a taken one 20. So
// everything that does not depend on the answer in flight is computed while it is on the way (the exact boundary while
// the cells' places are read, the reciprocal of the count while its power is), one branch leaves the straight line for
// everything that is rare, and what the next batch needs is requested a batch ahead. A boundary has one comparison per
// value: the first value on its upper side is the rounded midpoint or the one after it. Measured (us per batch,
// Gaussian values, one table of 32 levels, buckets of 128 / 352 / 512 / 1024 / 2048): 0.32 / 0.34 / 0.34 / 0.37 / 0.62,
// against 0.40 / 0.43 / 0.44 / 0.48 / 0.91 with barriers, 64-bit words in the cells, two rounded distances per value
// and a table of reciprocals; 6 bits, 1024: 0.58 -> 0.40; the 292 tables of the 350M model 507 -> 390 us. Up to 512
// values the chain binds, 770-830 cycles a batch with LDS in use for 150-340 of them. At 1024 (890 cycles, LDS in use
// for 540, half of these in bank conflicts) chain and producers are level: with seven, nine, ten, eleven, twelve and
// thirteen producers a batch of 544 takes 0.45, 0.46, 0.43, 0.40, 0.55, 0.50, one of 1024 0.39, 0.41, 0.39, 0.37, 0.41,
// 0.38 (12 waves are three to a SIMD, which more than eleven producers are not). At 2048 the sorting binds (1490
// cycles, LDS in use for 900), of which LDS holds room for eight slots. Tensors of few batches are bound by what a
// workgroup does before its first one, the table of powers above all, and by one workgroup of this size to a compute
// unit: 2000 tensors of one batch of 128 / 512 / 1024 / 2048, 5 bits, 8.7 / 26.7 / 32.6 / 53.3 us with barriers, 8.0 /
// 21.9 / 27.4 / 41.6 now, 300 of them 4.5 / 7.3 / 8.9 / 13.7 and 3.9 / 6.2 / 7.6 / 10.8.
//
// The boundary search needs levels that ascend by more than 2^-20 within [0, 1 + 2^-22] (then the comparison of the two
// rounded distances is monotone in the value and flips within 2^-22 of the midpoint, which is below 1) and cells that
// are not crowded. A batch for which that does not hold is assigned value by value, by the same wave.
// ---------------------------------------------------------------------------------------
// Shape of a workgroup: a producer sorts a batch of up to 64 * VPT values.
template <int BMAX, int C>
struct FitSlot;

template <int BITS, int VPT, int W>
struct FitShape {
    static_assert(W == 1, "a wave to a batch");
    static constexpr int kBucketMax = 64 * VPT;
    // Six producers for buckets of 129-256 and, with up to 8 levels, of 257-512: seven leave room for fewer workgroups
    // on a compute unit, and the chain is no faster with them. Eleven for 513-1024 (above), which makes tensors of one
    // batch 1-3 % slower than seven would; of the largest buckets LDS holds eight batches.
    static constexpr int kProducers = VPT == 16                             ? 11
                                      : VPT == 4 || (VPT == 8 && BITS <= 3) ? 6
                                                                            : 7;
    static constexpr int kSlots = VPT == 32 ? 8 : VPT == 16 ? 14 : 2 * kProducers;
    static_assert(kProducers <= kSlots, "a slot for every producer");
    static constexpr int kThreads = 64 * (kProducers + 1);  // and the consumer
    // About a cell per value (the middle of a Gaussian batch has two and a half to a cell), with more levels two cells:
    // a lane sees four or eight values from a group's start on at once, and one boundary that has more costs all of
    // them another read (1024, 5 bits: 0.52 us per batch with half the cells).
    static constexpr int kCells = VPT >= 16 ? 1024 : (BITS >= 5 ? 2 : 1) * kBucketMax;
    using Slot = FitSlot<kBucketMax, kCells>;
};

// Count and sum of a set of normalised values in one word: sum of at most 2^11 values of at most 2^32 + 2^10 below,
// count above.
constexpr int kFitCountShift = 48;
constexpr uint64_t kFitSumMask = (1ull << kFitCountShift) - 1;

// The normalised values are held in units of 2^-32, an exact scaling, so that their fixed-point form is a conversion.
constexpr float kFitUnit = 0x1p32f;

// What follows the values of a batch: above every boundary, as many as the consumer reads at once.
constexpr float kFitFiller = 2.0f * kFitUnit;
constexpr int kFitSpare = 20;

// z (units of 2^-32) as an integer, truncated, and a count of one. The conversion saturates from 1 on, where z is a
// whole number of units, 2^9 of them to a step of its last bit; below 1 it never gives all ones.
__device__ __forceinline__ uint64_t fit_word(float z) {
    const uint32_t fraction = (uint32_t)z;
    const bool one = fraction == ~0u;
    const uint32_t excess = (__float_as_uint(z) - __float_as_uint(kFitUnit)) << 9;
    return ((uint64_t)((1u << (kFitCountShift - 32)) + (one ? 1u : 0u)) << 32) | (one ? excess : fraction);
}

// A bucket's range of more than 2^126 has a subnormal reciprocal, off by up to 2^-150, and the largest of its
// normalised values can be 1 + 2^-23 or 1 + 2^-22; with any other range it is 1 at most (the product of a number and
// its rounded reciprocal is within 2^-24 of 1).
__device__ __forceinline__ bool fit_past_one(const MinMaxGrid& grid) {
    return grid.inv > 0.0f && grid.inv < 0x1p-126f;
}

// The cell of a value: C cells of equal width, what lies outside them in the first and the last. Monotone, and in range
// whatever the argument (the conversion saturates).
struct FitCells {
    float origin, per_unit;
};
template <int C>
__device__ __forceinline__ uint32_t fit_cell(float z, FitCells cells) {
    const uint32_t c = (uint32_t)fmaf(z, cells.per_unit, cells.origin);
    return c < (uint32_t)C ? c : (uint32_t)(C - 1);
}

// The same cells as the consumer asks for them, of a boundary halfway between two levels whose sum is s: the first
// cell that may hold values on both sides is that of s * half_unit + before, the one past the last that of s *
// half_unit + past. The margin of 2^-20 of the unit interval covers the 2^-22 within which the comparison flips and
// the roundings here and in fit_cell (each below 2^-23; `origin`, with whatever error, is the same in both).
struct FitBoundary {
    float half_unit, before, past;
};
__device__ __forceinline__ FitBoundary fit_boundary(FitCells cells) {
    const float margin = 0x1p-20f * cells.per_unit;
    return {0.5f * cells.per_unit, cells.origin - margin, cells.origin + margin + 1.0f};
}

// The cells for a batch: over its mean +- four times its mean magnitude, within its range [lo, hi]. That is the whole
// range for Gaussian weights; for heavy-tailed gradients it keeps the cells where the values are (a range stretched
// by one outlier would put most of a batch into a few cells).
template <int C>
__device__ __forceinline__ FitCells fit_cells(const MinMaxGrid& grid, float hi, float mean, float magnitude) {
    const float from = fmaxf(grid.lo, mean - 4.0f * magnitude);
    const float to = fminf(hi, mean + 4.0f * magnitude);
    const float width = (to - from) * grid.inv;
    const float per_unit = (float)C / width;
    const FitCells inner = {(grid.lo - from) * grid.inv * per_unit, per_unit};
    const FitCells all = {0.0f, (float)C};
    return width > 0x1p-20f && width <= 2.0f ? inner : all;
}

// Inclusive prefix sums over the lanes of a wave, of N values side by side.
template <int CTRL, int ROWS, int N>
__device__ __forceinline__ void fit_scan_step(uint32_t (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v[i], CTRL, ROWS, 0xF, false);
}
template <int N>
__device__ __forceinline__ void fit_wave_scan(uint32_t (&v)[N]) {
    fit_scan_step<0x111, 0xF>(v);  // row_shr:1, 2, 4, 8: within rows of 16 lanes
    fit_scan_step<0x112, 0xF>(v);
    fit_scan_step<0x114, 0xF>(v);
    fit_scan_step<0x118, 0xF>(v);
    fit_scan_step<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    fit_scan_step<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
}

// Halves of a word of count and sum. Additions are of whole words (one instruction, with halves in registers of their
// own two and a wait between them), so what the halves are put together to is hidden from the compiler.
struct FitWord {
    uint32_t low, high;
};
__device__ __forceinline__ FitWord fit_halves(uint64_t v) { return {(uint32_t)v, (uint32_t)(v >> 32)}; }
__device__ __forceinline__ uint64_t fit_whole(FitWord v) {
    uint64_t w = ((uint64_t)v.high << 32) | v.low;
    asm("" : "+v"(w));
    return w;
}

// Sum over the lanes l, l + 64/S, l + 2 * 64/S, ... (S = 1, 2, 4). The exchanges by hand: both copies, then one wait
// for both (the compiler waits for each).
template <int S>
__device__ __forceinline__ uint64_t fit_sum_subs(uint64_t sum) {
    if constexpr (S >= 2) {
        FitWord v = fit_halves(sum), w;
        asm("v_mov_b32 %2, %0\n\tv_mov_b32 %3, %1\n\ts_nop 1\n\tv_permlane32_swap_b32 %0, %2\n\t"
            "v_permlane32_swap_b32 %1, %3" : "+v"(v.low), "+v"(v.high), "=&v"(w.low), "=&v"(w.high));
        sum = fit_whole(v) + fit_whole(w);
    }
    if constexpr (S >= 4) {
        FitWord v = fit_halves(sum), w;
        asm("v_mov_b32 %2, %0\n\tv_mov_b32 %3, %1\n\ts_nop 1\n\tv_permlane16_swap_b32 %0, %2\n\t"
            "v_permlane16_swap_b32 %1, %3" : "+v"(v.low), "+v"(v.high), "=&v"(w.low), "=&v"(w.high));
        sum = fit_whole(v) + fit_whole(w);
    }
    return sum;
}

// Keeps the compiler from reordering LDS accesses of one wave, which are processed in order.
__device__ __forceinline__ void fit_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

template <int BMAX>
struct FitPowers : FitChain<BMAX> {
    using Chain = FitChain<BMAX>;
    using Chain::kFine;
    double fine[kFine + 1];  // 1 - (1-lr)^c
    typename Chain::Coarse coarse;

    __device__ FitFilled start(int lane) {
        if (lane == 0) fine[0] = 0.0;
        return {0, 1.0};
    }

    __device__ __forceinline__ void extend(FitFilled& f, double one_minus, int lane) {
        Chain::extend(f, one_minus, lane, [&](uint32_t c) -> double& { return fine[c]; }, coarse);
    }

    // Where the level lands after the c values (at most kFine) of fixed-point sum `total` that are its own, given
    // 1 - (1-lr)^c. Without values it stays, whatever it holds. Everything but the last three steps is computed while
    // that power is on its way, the reciprocal of the count among it.
    static __device__ __forceinline__ float step(float level, uint32_t c, uint64_t total, double moved) {
        // total / c rounded once: r, the approximate reciprocal, is off by at most 2^-23 of itself, so a by 2^-22 and,
        // corrected once, by 2^-44, 2^9 ulp; its remainder is exact (c is at most 2^10: below 2^20 ulp), and the
        // quotient corrected again is within 2^-13 ulp of t / c, which, t * 2^32 and c being integers of at most 2^43
        // and 2^10, is never closer than 2^-11 ulp to a rounding boundary without being a binary64 number itself. (The
        // first remainder, below 2^42 ulp, is exact too.) Without values it is not used.
        const double n = (double)c;
        const double r = (double)__builtin_amdgcn_rcpf((float)c);
        const double q = (double)level;
        const double t = fma((double)(uint32_t)total, 0x1p-32, (double)(uint32_t)(total >> 32));
        const double rough = t * r;
        const double a = fma(fma(-rough, n, t), r, rough);
        const double mean = fma(fma(-a, n, t), r, a);
        return c == 0u ? level : (float)(q - moved * (q - mean));
    }

    // The same for any c.
    __device__ float step_any(float level, uint32_t c, uint64_t total, double one_minus) const {
        if (c <= (uint32_t)kFine) return step(level, c, total, fine[c]);
        return Chain::step_past_fine(level, c, total, one_minus, coarse);
    }
};

// A batch as the consumer reads it: the values grouped by cell (ascending cells, any order within one), the place of
// every cell's first value, and count and sum of the values before every fourth one. The place of cell C is
// the number of values rounded up to a multiple of four; the word before that place is that of all values.
template <int BMAX, int C>
struct alignas(16) FitSlot {
    static constexpr int kValues = BMAX;
    static constexpr int kGroups = BMAX / 4;
    uint32_t cell[C + 1];  // the last one: the end
    uint32_t ready;        // the batch's number + 1
    FitBoundary boundary;
    uint32_t unused[3];
    uint64_t before[kGroups + 2];
    float z[BMAX + kFitSpare];  // units of 2^-32, grouped by cell, kFitSpare fillers past the last one
};

// Groups of four values that a lane reads at once: two where a level has one lane (us per batch of 128 / 1024, one
// group and two: 7 bits 0.74 / 0.82 and 0.54 / 0.64, 8 bits 1.25 / 1.43 and 0.94 / 1.19; 5 bits, two lanes to a level,
// 0.33 / 0.37 and 0.36 / 0.40).
template <int BITS>
constexpr int kFitGroups = FitLanes<BITS>::S == 1 ? 2 : 1;

// What the consumer knows of the batch to come.
struct FitNext {
    FitBoundary boundary;
    uint32_t ready;
};
template <typename Slot>
__device__ __forceinline__ FitNext fit_next(const Slot& slot) {
    FitNext next;
    next.ready = __hip_atomic_load(&slot.ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    fit_order();
    next.boundary = slot.boundary;
    return next;
}

// The lanes with a level that is not in [0, 1]. One that is stays within [0, 1 + 2^-22], as far as the values reach
// (fit_past_one), towards a mean of which it moves.
template <int M>
__device__ __forceinline__ uint64_t fit_outside(const float (&lv)[M]) {
    uint64_t outside = 0;
#pragma unroll
    for (int i = 0; i < M; ++i) outside |= __builtin_amdgcn_ballot_w64(!(lv[i] >= 0.0f && lv[i] <= 1.0f));
    return outside;
}

// One batch of the chain. lv[i]: the lane's levels, level M * (lane mod (64 / S)) + i, updated; next: what is known of
// the batch, and then of the one in next_slot; outside: the lanes with a level that is not in [0, 1]; boundaries: those
// whose last level has one above it; not_first: 0 in the lanes of the first level; crowded: values in a boundary's
// cells from which the plain assignment is faster; count(): the batch's values; done(): the slot has been read;
// lv_shared, acc: K entries of LDS each, for batches that are assigned value by value.
template <int BITS, typename Slot, typename Powers, int C, typename Count, typename Done>
__device__ __forceinline__ void fit_batch(const Slot& slot, const Slot& next_slot, FitNext& next, uint64_t& outside,
                                          uint64_t boundaries, uint32_t not_first,
                                          uint32_t crowded, int bucket, Count count, Done done, Powers& powers,
                                          FitFilled& filled, double one_minus, float (&lv)[FitLanes<BITS>::M],
                                          float* lv_shared, uint64_t* acc, int lane) {
    constexpr int K = FitLanes<BITS>::K, S = FitLanes<BITS>::S, M = FitLanes<BITS>::M, G = kFitGroups<BITS>;
    static_assert(4 * S * G <= kFitSpare - 4, "reads past the last value");
    const int sub = S > 1 ? lane / (64 / S) : 0;
    const int k0 = S > 1 ? lane % (64 / S) : lane;
    const FitBoundary boundary = next.boundary;
    const float* values = slot.z + 4 * sub;
    float threshold[M];  // the values below it are on the lower one's side
    uint32_t pos[M], end[M];
    uint64_t narrow = 0;
    float upper_level[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const bool inner = M * k0 + i < K - 1;
        upper_level[i] = i + 1 < M ? lv[i + 1 < M ? i + 1 : 0] : __uint_as_float(next_lane(__float_as_uint(lv[0])));
        // a lane past the last boundary: the end
        float both = lv[i] + upper_level[i];
        if (M == 1) {  // the move is folded into this addition, as the sum is its only use
            float again = lv[i];
            asm volatile("" : "+v"(again));
            both = lv[i] + __uint_as_float(next_lane(__float_as_uint(again)));
        }
        const float from = __builtin_amdgcn_fmed3f(fmaf(both, boundary.half_unit, boundary.before),
                                                   inner ? 0.0f : (float)C, inner ? (float)(C - 1) : (float)C);
        const float to = __builtin_amdgcn_fmed3f(fmaf(both, boundary.half_unit, boundary.past),
                                                 inner ? 1.0f : (float)C, (float)C);
        pos[i] = slot.cell[(uint32_t)from];
        end[i] = slot.cell[(uint32_t)to];
    }
    next = fit_next(next_slot);
#pragma unroll
    for (int i = 0; i < M; ++i) {
        // The first value that is closer to the upper level is the rounded midpoint or the one after it: the midpoint
        // is off by half a step, so that a step further the distances differ by a step or more, and of them only the
        // one to a level below half the value is rounded, by half a step.
        const float mid = 0.5f * (lv[i] + upper_level[i]);
        threshold[i] = kFitUnit * __uint_as_float(__float_as_uint(mid) +
                                                  (fabsf(mid - upper_level[i]) < fabsf(mid - lv[i]) ? 0u : 1u));
        asm volatile("" : "+v"(threshold[i]));  // here, while the places are on their way
        narrow |= __builtin_amdgcn_ballot_w64(!(upper_level[i] - lv[i] > 0x1p-20f)) &
                  (i + 1 < M ? ~0ull : boundaries);
    }
    uint64_t upto[M];  // count and sum of the values of levels 0 .. k
    f4 z[M][G];
    uint64_t rare = outside | narrow;
    uint32_t group[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
        group[i] = pos[i] & ~3u;
#pragma unroll
        for (int g = 0; g < G; ++g) z[i][g] = *reinterpret_cast<const f4*>(&values[group[i] + 4u * S * g]);
        upto[i] = slot.before[group[i] >> 2];
        rare |= __builtin_amdgcn_ballot_w64(end[i] > group[i] + 4u * S * G);
    }
    // count and sum of those of four values that are on the lower level's side: below 1 (the boundary is), so 32 bits
    // hold them. Values past the boundary's cells may be among the four, and fillers past the
    // last one: above the boundary.
    auto below_of = [&](f4 v, float t) -> uint64_t {
        uint64_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool lower = v[u] < t;
            const uint32_t fixed = (uint32_t)v[u];
            w[u] = ((uint64_t)(lower ? 1u << (kFitCountShift - 32) : 0u) << 32) | (lower ? fixed : 0u);
        }
        uint64_t left = w[0] + w[1], right = w[2] + w[3];
        asm("" : "+v"(left), "+v"(right));  // side by side
        return left + right;
    };
    bool by_value = false;
    if (__builtin_expect(rare != 0, 0)) {
        uint64_t plain = outside | narrow;
#pragma unroll
        for (int i = 0; i < M; ++i)
            plain |= __builtin_amdgcn_ballot_w64(end[i] - group[i] > crowded && end[i] > group[i]);
        by_value = plain != 0;
        if (!by_value) {  // the groups that follow, of all the lane's levels side by side
            uint64_t more[M] = {};
            for (uint32_t next_group = 4u * S * G;; next_group += 4u * S) {
                uint64_t left = 0;
                f4 v[M];
#pragma unroll
                for (int i = 0; i < M; ++i) {
                    const uint32_t p = group[i] + next_group;
                    left |= __builtin_amdgcn_ballot_w64(p < end[i]);
                    v[i] = *reinterpret_cast<const f4*>(&values[p < end[i] ? p : group[i]]);
                }
                if (left == 0) break;
#pragma unroll
                for (int i = 0; i < M; ++i) {
                    const uint64_t w = below_of(v[i], threshold[i]);
                    more[i] += group[i] + next_group < end[i] ? w : 0ull;
                }
            }
#pragma unroll
            for (int i = 0; i < M; ++i) upto[i] += fit_sum_subs<S>(more[i]);
        }
    }
    FitWord own[M];
    if (__builtin_expect(!by_value, 1)) {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            uint64_t below = below_of(z[i][0], threshold[i]);
#pragma unroll
            for (int g = 1; g < G; ++g) below += below_of(z[i][g], threshold[i]);
            upto[i] += fit_sum_subs<S>(below);
        }
#pragma unroll
        for (int i = 0; i < M; ++i) {
            if (i > 0) {
                own[i] = fit_halves(upto[i] - upto[i > 0 ? i - 1 : 0]);
                continue;
            }
            const FitWord highest = fit_halves(upto[M - 1]);
            FitWord previous = {previous_lane(highest.low), previous_lane(highest.high)};
            if (S > 1) previous = {previous.low & not_first, previous.high & not_first};
            // not folded into the subtraction: v_subrev_u32 with a DPP operand gave the negative difference here
            asm volatile("" : "+v"(previous.low), "+v"(previous.high));
            own[i] = fit_halves(upto[i] - (((uint64_t)previous.high << 32) | previous.low));
        }
    } else {
        fit_by_value<BITS>(
            count(), lv, sub == 0, [&](int i) { return M * k0 + i; },
            [&](int p) { return slot.z[p] * (1.0f / kFitUnit); }, [](float z) { return fit_word(z * kFitUnit); },
            [&](int i, uint64_t word) { own[i] = fit_halves(word); }, lv_shared, acc, lane);
    }
    // the powers are requested before it is known whether the table holds them: the answer comes while they are on
    // the way
    uint32_t c[M], most = 0;
    double moved[M];
    auto request = [&] {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            if constexpr (Powers::kFine == Slot::kValues) {
                // eight bytes for every one of the count, the upper half of the word's upper half, in one instruction
                static_assert(kFitCountShift == 48 && sizeof(double) == 8, "place of the count");
                uint32_t at;
                asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
                    : "=v"(at) : "v"(3u), "v"(own[i].high));
                moved[i] = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(powers.fine) + at);
            } else {
                moved[i] = powers.fine[c[i] < (uint32_t)Powers::kFine ? c[i] : (uint32_t)Powers::kFine];
            }
        }
    };
#pragma unroll
    for (int i = 0; i < M; ++i) {
        c[i] = own[i].high >> (kFitCountShift - 32);
        most = c[i] > most ? c[i] : most;
    }
    request();
    done();
    next.ready = __builtin_amdgcn_readfirstlane(next.ready);
    if (filled.count < bucket) {
        while (__builtin_expect(__builtin_amdgcn_ballot_w64(most > (uint32_t)filled.count) != 0, 0)) {
            powers.extend(filled, one_minus, lane);
            request();
        }
    }
    if (Powers::kFine == Slot::kValues ||
        __builtin_expect(__builtin_amdgcn_ballot_w64(most > (uint32_t)Powers::kFine) == 0, 1)) {
#pragma unroll
        for (int i = 0; i < M; ++i) lv[i] = Powers::step(lv[i], c[i], fit_whole(own[i]) & kFitSumMask, moved[i]);
    } else {
#pragma unroll
        for (int i = 0; i < M; ++i) lv[i] = powers.step_any(lv[i], c[i], fit_whole(own[i]) & kFitSumMask, one_minus);
    }
    if (__builtin_expect(outside != 0, 0)) outside = fit_outside<M>(lv);
}

template <int BITS, int VPT, int W>
__global__ void __launch_bounds__((FitShape<BITS, VPT, W>::kThreads)) fit_levels_kernel(const FitParams p) {
    using Shape = FitShape<BITS, VPT, W>;
    using Slot = typename Shape::Slot;
    constexpr int C = Shape::kCells, P = Shape::kProducers, K = 1 << BITS;
    constexpr uint32_t kSlots = Shape::kSlots;
    constexpr int M = FitLanes<BITS>::M, S = FitLanes<BITS>::S;
    __shared__ Slot slots[kSlots];
    typedef FitPowers<Shape::kBucketMax> Powers;
    __shared__ Powers powers;
    __shared__ float lv_shared[K];
    __shared__ uint64_t acc[K];
    __shared__ uint32_t consumed[64];  // batches that the consumer has read, one copy for every lane
    __shared__ uint32_t nowhere[64];   // where lanes without a value count and write
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
    const double one_minus = 1.0 - (double)p.lr;
    if (threadIdx.x < 64) consumed[threadIdx.x] = 0;
    if (threadIdx.x < kSlots) slots[threadIdx.x].ready = 0;
    __syncthreads();  // the only one: from here on a wave waits for the words that it needs

    if (wave == Shape::kProducers) {
        __builtin_amdgcn_s_setprio(3);
        float lv[M];
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = M * (S > 1 ? lane % (64 / S) : lane) + i;
            lv[i] = k < K ? levels[k] : 0.0f;
        }
        FitFilled filled = powers.start(lane);
        // while the producers sort the first round: up to three times the mean count, which the fullest level of a
        // Gaussian batch on the uniform table does not reach; all of them for the smallest buckets
        while (filled.count < Powers::kFine && (Powers::kFine <= 256 || filled.count * K < 3 * B))
            powers.extend(filled, one_minus, lane);
        // values in a boundary's cells from which the plain assignment of the batch is faster
        const uint32_t crowded = (uint32_t)(B * 4 * S / (48 * M)) + 64u;
        uint64_t outside = fit_outside<M>(lv);
        // the last levels' lanes have no boundary above them, the first level's nothing before
        uint64_t boundaries = __builtin_amdgcn_ballot_w64(M * (S > 1 ? lane % (64 / S) : lane) + M - 1 < K - 1);
        asm volatile("" : "+s"(boundaries));  // kept, not asked again
        const uint32_t not_first = lane % (64 / S) == 0 ? 0u : ~0u;
        FitNext next;
        auto walk = [&](uint64_t j, uint32_t slot, uint32_t following) {
            auto done = [&] {
                fit_order();
                __hip_atomic_store(&consumed[lane], (uint32_t)j + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            fit_batch<BITS, Slot, Powers, C>(slots[slot], slots[following], next, outside, boundaries, not_first,
                                             crowded, B, [&] { return batch_size(j); }, done, powers, filled,
                                             one_minus, lv, lv_shared, acc, lane);
        };
        auto look = [&](uint32_t slot) {
            next = fit_next(slots[slot]);
            next.ready = __builtin_amdgcn_readfirstlane(next.ready);
        };
        uint32_t slot = 0;
        look(0);
        for (uint64_t j = 0; j < num_batches; ++j) {
            while (__builtin_expect(next.ready != (uint32_t)j + 1u, 0)) look(slot);
            fit_order();
            const uint32_t following = slot + 1 < kSlots ? slot + 1 : 0;
            walk(j, slot, following);
            slot = following;
        }
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = M * (S > 1 ? lane % (64 / S) : lane) + i;
            if ((S == 1 || lane < 64 / S) && k < K) levels[k] = lv[i];
        }
    } else {
        // Lanes past the end of a batch fetch its last value, which changes no minimum or maximum, and enter nothing.
        float next[VPT];
        auto fetch = [&](uint64_t j) {
            const int m = batch_size(j);
            const float* src = v + j * (uint64_t)B;
            if (m == Shape::kBucketMax) {
#pragma unroll
                for (int q = 0; q < VPT; ++q) next[q] = src[(uint32_t)(lane + 64 * q)];
            } else {
#pragma unroll
                for (int q = 0; q < VPT; ++q) {
                    const int i = lane + 64 * q;
                    next[q] = src[(uint32_t)(i < m ? i : m - 1)];
                }
            }
        };
        uint32_t place_of = (uint32_t)wave;  // the batch's slot
        // One batch; `full`: a value in every lane, so that nothing asks which are there.
        auto sort = [&](uint64_t j, auto full_batch) {
            constexpr bool full = decltype(full_batch)::value;
            const int m = full ? Shape::kBucketMax : batch_size(j);
            auto there = [&](int q) { return full || lane + 64 * q < m; };
            Slot& slot = slots[place_of];
            constexpr int kSampled = VPT >= 8 ? 4 : 1;  // every fourth value is enough to place the cells
            float z[VPT];
            float lo = next[0], hi = next[0], sum = 0.0f, absolute = 0.0f;
#pragma unroll
            for (int q = 0; q < VPT; ++q) {
                z[q] = next[q];
                lo = fminf(lo, z[q]);
                hi = fmaxf(hi, z[q]);
                if (q % kSampled == 0) {
                    sum += z[q];
                    absolute += fabsf(z[q]);
                }
            }
            if (j + P < num_batches) fetch(j + P);  // in flight while this batch is sorted
            lo = group_min<64>(lo);
            hi = group_max<64>(hi);
            sum = fit_wave_sum(sum);
            absolute = fit_wave_sum(absolute);
            // the slot is free once the consumer has read the batch that it held
            while ((uint32_t)j - __builtin_amdgcn_readfirstlane(__hip_atomic_load(
                                     &consumed[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) >= kSlots)
                __builtin_amdgcn_s_sleep(1);
            fit_wave_sync();
#pragma unroll
            for (int c0 = 0; c0 < C; c0 += 256) {
                const int c = c0 + 4 * lane;
                if (C % 256 == 0 || c < C) *reinterpret_cast<u4*>(&slot.cell[c]) = u4{0u, 0u, 0u, 0u};
            }
            fit_wave_sync();
            const MinMaxGrid grid = make_minmax_grid(lo, hi, 1.0f, false);
            const bool past_one = __builtin_amdgcn_readfirstlane(fit_past_one(grid)) != 0;
            const FitCells cells = fit_cells<C>(grid, hi, sum * ((float)kSampled / (64 * VPT)),
                                                absolute * ((float)kSampled / (64 * VPT)));
            uint32_t* cell[VPT];
            uint32_t held[VPT];  // the values that the cell held before this one came
            // Rows of a wave's values eight at a time, so that what a short batch does not have is left out and the
            // rest is straight-line code: a lane without a value uses words of its own.
            auto rows = [&](auto each) {
#pragma unroll
                for (int q0 = 0; q0 < VPT; q0 += 8)
                    if (full || 64 * q0 < m) {
#pragma unroll
                        for (int q = q0; q < q0 + 8 && q < VPT; ++q) each(q);
                    }
            };
            rows([&](int q) {
                z[q] = (z[q] - grid.lo) * grid.inv;
                cell[q] = there(q) ? &slot.cell[fit_cell<C>(z[q], cells)] : &nowhere[lane];
                z[q] *= kFitUnit;
                held[q] = fit_add(cell[q], 1u);
            });
            fit_wave_sync();
            // lane l has cells 4l .. 4l + 3 of every row of 256
            constexpr int kCellRows = C >= 256 ? C / 256 : 1;
            u4 own[kCellRows];
            uint32_t sum4[kCellRows], upto[kCellRows], base_cell = 0;
#pragma unroll
            for (int i = 0; i < kCellRows; ++i) {
                const int c = 4 * (64 * i + lane);
                own[i] = C >= 256 || c < C ? *reinterpret_cast<const u4*>(&slot.cell[c]) : u4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int i = 0; i < kCellRows; ++i) upto[i] = sum4[i] = (own[i][0] + own[i][1]) + (own[i][2] + own[i][3]);
            fit_wave_scan(upto);
#pragma unroll
            for (int i = 0; i < kCellRows; ++i) {
                const int c = 4 * (64 * i + lane);
                u4 at;
                at[0] = base_cell + upto[i] - sum4[i];
                at[1] = at[0] + own[i][0];
                at[2] = at[1] + own[i][1];
                at[3] = at[2] + own[i][2];
                if (C >= 256 || c < C) *reinterpret_cast<u4*>(&slot.cell[c]) = at;
                base_cell += (uint32_t)__builtin_amdgcn_readlane((int)upto[i], 63);
            }
            if (lane == 0) slot.cell[C] = (uint32_t)(m + 3) & ~3u;
            fit_wave_sync();
            // all places requested before the first one is waited for
            rows([&](int q) { held[q] += *cell[q]; });
            rows([&](int q) {
                float* at = there(q) ? &slot.z[held[q]] : reinterpret_cast<float*>(&nowhere[lane]);
                *at = z[q];
            });
            if (lane < kFitSpare) slot.z[m + lane] = kFitFiller;
            fit_wave_sync();
            // Count and sum before every group of four values, rows of 64 groups side by side; the sums of the
            // values' upper and lower 16 bits apart, so that 32 bits hold them. A value of 1 (the conversion saturates)
            // is one short here, one past 1 by more: they are above every boundary, so that only the word of all values
            // has to know.
            constexpr int kRows = VPT >= 4 ? VPT / 4 : 1;
            constexpr bool kHalf = VPT < 4;  // half a row
            uint32_t incl[2 * kRows], row[2 * kRows], ones = 0;
            const uint32_t crest = slot.cell[fit_cell<C>(1.0f, cells)];  // where the values of the cell of 1 start
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                const int g = 64 * i + (kHalf ? lane & 31 : lane);
                const f4 four = *reinterpret_cast<const f4*>(&slot.z[4 * g]);
                uint32_t low = 0, high = 0;
                uint32_t fixed[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    fixed[u] = full || 4 * g + u < m ? (uint32_t)four[u] : 0u;
                    low += fixed[u] & 0xFFFFu;
                    high += fixed[u] >> 16;
                }
                if ((uint32_t)__builtin_amdgcn_readfirstlane((int)crest) < 256u * (uint32_t)(i + 1)) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool one = fixed[u] == ~0u && (!kHalf || lane < 32);
                        ones += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(one));
                    }
                }
                incl[2 * i] = row[2 * i] = low;
                incl[2 * i + 1] = row[2 * i + 1] = high;
            }
            fit_wave_scan(incl);
            constexpr int kLast = kHalf ? 31 : 63;
            auto last = [&](uint32_t x) { return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)x, kLast); };
            uint64_t base = 0;
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                const int g = 64 * i + lane;
                const uint32_t c = full || 4 * g < m ? (uint32_t)(4 * g) : (uint32_t)m;
                const uint64_t before =
                    base + (incl[2 * i] - row[2 * i]) + ((uint64_t)(incl[2 * i + 1] - row[2 * i + 1]) << 16);
                if (!kHalf || lane < 32) slot.before[g] = before + ((uint64_t)c << kFitCountShift);
                base += last(incl[2 * i]) + (last(incl[2 * i + 1]) << 16);
            }
            if (__builtin_expect(past_one, 0)) {  // what the conversion left out of values past 1
                uint32_t excess[1] = {0};
#pragma unroll 1
                for (int i = lane; i < m; i += 64)
                    excess[0] += slot.z[i] > kFitUnit ? (uint32_t)(slot.z[i] - kFitUnit) : 0u;
                fit_wave_scan(excess);
                base += (uint32_t)__builtin_amdgcn_readlane((int)excess[0], 63);
            }
            fit_wave_sync();
            if (lane == 0) {
                slot.before[(m + 3) >> 2] = base + ones + ((uint64_t)m << kFitCountShift);  // of all values
                slot.boundary = fit_boundary(cells);
                fit_order();
                __hip_atomic_store(&slot.ready, (uint32_t)j + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        };
        if ((uint64_t)wave < num_batches) fetch((uint64_t)wave);
        for (uint64_t j = (uint64_t)wave; j < num_batches; j += P) {
            if (batch_size(j) == Shape::kBucketMax) sort(j, std::true_type{});
            else sort(j, std::false_type{});
            place_of = place_of + P < kSlots ? place_of + P : place_of + P - kSlots;
        }
    }
}

}  // namespace qsdp
