// Level fitting for buckets of more than 2048 values (see qsdp_fit_kernel.hpp for the smaller ones and the definition).
// The form of a batch (units of the values, cells, count and sum in a word) is this kernel's own.
#pragma once

#include "qsdp_fit_common.hpp"

namespace qsdp {
namespace fit_rounds {

// ---------------------------------------------------------------------------------------
// As in qsdp_fit_kernel.hpp producer waves sort the coming batches into cells and one consumer wave walks the chain,
// but a team of W = 4 or 8 waves sorts a batch and all waves meet at barriers, four to a batch; P = 8 / W batches make
// a round, the consumer walks those of the round before, the slots are double-buffered. The sums of the values before a
// cell come from the sort's own counting (count and sum in one 64-bit LDS atomic per value), which needs two passes
// less than the other kernel's sums over groups of four: that is what counts where a batch has a compute unit's LDS to
// itself and its passes come one after the other (us per batch, 5 bits, buckets of 4096 / 8192: 1.73 / 3.25, and 1.82 /
// 4.77 in the other kernel's way with teams of two and four waves; a bucket of 2048 0.91 and 0.62).
// ---------------------------------------------------------------------------------------
// Shape of a workgroup: W waves to a batch of up to 64 * W * VPT values.
template <int BMAX, int C>
struct FitSlot;

template <int BITS, int VPT, int W>
struct FitShape {
    static constexpr int kBucketMax = 64 * W * VPT;
    static constexpr int kBatches = 8 / W;           // P, batches per round
    static constexpr int kProducers = kBatches * W;  // producer waves; the consumer is one more
    static constexpr int kThreads = 64 * (kProducers + 1);
    static constexpr int kBarriers = 4;  // per round
    static constexpr int kCells = 1024;
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

// The powers beside the reciprocals of the counts, which are the producers' work while their first loads are on the
// way.
template <int BMAX>
struct FitPowers : FitChain<BMAX> {
    using Chain = FitChain<BMAX>;
    using Chain::kFine;
    struct Entry {
        double moved, reciprocal;  // 1 - (1-lr)^c, 1 / c
    };
    Entry fine[kFine + 1];
    typename Chain::Coarse coarse;

    __device__ void fill_reciprocals(int top, int thread, int threads) {
        for (int c = thread; c <= kFine && c <= top; c += threads) fine[c].reciprocal = 1.0 / (double)(c > 0 ? c : 1);
    }

    __device__ FitFilled start(int lane) {
        if (lane == 0) fine[0].moved = 0.0;
        return {0, 1.0};
    }

    __device__ __forceinline__ void extend(FitFilled& f, double one_minus, int lane) {
        Chain::extend(f, one_minus, lane, [&](uint32_t c) -> double& { return fine[c].moved; }, coarse);
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
        return Chain::step_past_fine(level, c, total, one_minus, coarse);
    }
};

// A batch as the consumer reads it: the values grouped by cell (ascending cells, any order within one), and for every
// cell count and sum of the values in the cells before it; cell C: of all values.
// The prefix sum gives a lane kOwn cells in a row; one word of padding after each of these runs keeps the lanes off
// one another's banks (without it all 64 lanes meet in two banks: 0.15 us more per batch of 1024).
template <int BMAX, int C>
struct FitSlot {
    static constexpr int kOwn = C / 64;
    static __device__ __forceinline__ uint32_t at(uint32_t c) { return c + c / kOwn; }
    uint64_t cell[C + 64 + 1];  // cell c at at(c)
    float z[BMAX + kFitSpare];  // grouped by cell, kFitSpare fillers past the last one
    FitCells cells;
};

// One batch of the chain. lv[i]: the lane's levels, level 64 * i + lane mod (64 / S), updated. lv_shared, acc: K
// entries of LDS each, for batches that are assigned value by value.
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
            const float following =
                __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lv[i + 1 < M ? i + 1 : 0]), 0));
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
        fit_by_value<BITS>(
            m, lv, sub == 0, [&](int i) { return 64 * i + k0; }, [&](int p) { return slot.z[p]; },
            [](float z) { return (1ull << kFitCountShift) | fit_fixed(z); },
            [&](int i, uint64_t word) { own[i] = word; }, lv_shared, acc, lane);
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
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(most > (uint32_t)Powers::kFine) == 0, 1)) {
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
        // Gaussian batch on the uniform table does not reach
        while (filled.count < Powers::kFine && filled.count * K < 3 * B)
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
                for (int b = 0; b < Shape::kBarriers / P; ++b) __syncthreads();
            }
        }
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const int k = 64 * i + (S > 1 ? lane % (64 / S) : lane);
            if ((S == 1 || lane < 64 / S) && k < K) levels[k] = lv[i];
        }
    } else {
        auto team_sync = [] { __syncthreads(); };  // between the passes of a team
        // a producer: batch r * P + team in round r, this wave's 1/W of it; nothing but the barriers past the last one.
        // Lanes past the end of a batch fetch its last value, which changes no minimum or maximum, and enter nothing.
        const int team = wave / W, part = wave % W;
        const int scanner = W == 4 ? team : 0;  // of the team's waves: on another SIMD for every team
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
            const MinMaxGrid grid = make_minmax_grid(lo, hi, 1.0f, false);
            const FitCells cells = fit_cells<C>(grid, hi, sum * (1.0f / (64 * W * VPT)),
                                                absolute * (1.0f / (64 * W * VPT)));
            uint32_t cell[VPT];
            // the cell's word before this value came (both halves used: half of one dropped costs a wait)
            uint64_t held[VPT];
            auto enter = [&](int q) {
                z[q] = (z[q] - grid.lo) * grid.inv;
                cell[q] = Slot::at(fit_cell<C>(z[q], cells));
                held[q] = fit_add<uint64_t>(&slot.cell[cell[q]], (1ull << kFitCountShift) | fit_fixed(z[q]));
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

}  // namespace fit_rounds
}  // namespace qsdp
