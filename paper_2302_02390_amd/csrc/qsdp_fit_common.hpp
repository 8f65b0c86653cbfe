// What the two kernels of the level fit share: qsdp_fit_kernel.hpp, a wave to a batch, and qsdp_fit_rounds.hpp, a team
// of waves. A translation unit includes one of them.
#pragma once

#include "qsdp_params.hpp"

namespace qsdp {

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

// Adds to a word in LDS and returns what it held. Relaxed: the callers put their own fences, and an ordered atomic
// would wait for each one before the next.
template <typename T>
__device__ __forceinline__ T fit_add(T* word, T v) {
    return __hip_atomic_fetch_add(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// LDS traffic of one wave is processed in order; this keeps the compiler from reordering it.
__device__ __forceinline__ void fit_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (1 - lr)^c by repeated multiplication, the order in which c single steps compound, for c up to the bucket size:
// every power up to kFine, beyond that every kStep-th. The multiplications are a serial chain (about 8 ns each), so
// the consumer extends it as the counts ask for it: most counts are a small share of a bucket, and a tensor of few
// batches would wait for powers that it never reads.
struct FitFilled {
    int count;    // the powers of counts up to this one can be read
    double keep;  // where the chain stands
};
template <int BMAX>
struct FitChain {
    static constexpr int kFine = BMAX < 1024 ? BMAX : 1024, kStep = 16, kCoarse = (BMAX - kFine) / kStep + 1;
    static_assert(kFine % 64 == 0, "grows by 64");
    typedef double Coarse[kCoarse];

    // The next 64 powers, 1 - (1-lr)^c in fine(c), or the next 16 of every kStep-th, (1-lr)^c (one wave; the chain and
    // its stores in one lane).
    template <typename Fine>
    static __device__ __forceinline__ void extend(FitFilled& f, double one_minus, int lane, Fine fine, Coarse& coarse) {
        double keep = f.keep;
        if (f.count < kFine) {
            if (lane == 0) {
                uint32_t first = (uint32_t)f.count + 1u;
                asm volatile("" : "+v"(first));  // one address register, the stores' offsets in the instructions
#pragma unroll 16
                for (int i = 0; i < 64; ++i) {
                    keep *= one_minus;
                    fine(first + i) = keep;
                }
            }
            fit_wave_sync();
            double& mine = fine(f.count + 1 + lane);
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

    // Where the level lands after the c values, more than kFine, of fixed-point sum `total` that are its own.
    static __device__ __forceinline__ float step_past_fine(float level, uint32_t c, uint64_t total, double one_minus,
                                                           const Coarse& coarse) {
        const int k = ((int)c - kFine) / kStep;
        double keep = coarse[k];
        for (int i = kFine + k * kStep; i < (int)c; ++i) keep *= one_minus;
        const double q = (double)level;
        const double mean = ((double)total / (double)c) * (1.0 / 4294967296.0);
        return c == 0u ? level : (float)(q - (1.0 - keep) * (q - mean));
    }
};

// How the levels of a table are shared among the lanes: S lanes to a level or M levels to a lane.
template <int BITS>
struct FitLanes {
    static constexpr int K = 1 << BITS;
    static constexpr int S = K <= 16 ? 4 : K <= 32 ? 2 : 1;
    static constexpr int M = K <= 64 ? 1 : K / 64;
};

// A batch value by value against the table in LDS: level_of(i) is the lane's level i (of M), value(p) value p of m,
// word(z) count and sum of a value; done(i, word) gets those of level i. lv_shared, acc: K entries of LDS each.
template <int BITS, typename LevelOf, typename Value, typename Word, typename Done>
__device__ __forceinline__ void fit_by_value(int m, const float (&lv)[FitLanes<BITS>::M], bool first_of_level,
                                             LevelOf level_of, Value value, Word word, Done done, float* lv_shared,
                                             uint64_t* acc, int lane) {
    constexpr int K = FitLanes<BITS>::K, M = FitLanes<BITS>::M;
    fit_wave_sync();
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const int k = level_of(i);
        if (first_of_level && k < K) {
            lv_shared[k] = lv[i];
            acc[k] = 0;
        }
    }
    fit_wave_sync();
    for (int p = lane; p < m; p += 64 * 4) {  // four values a lane at once: the searches' LDS reads overlap
        float z[4];
        int k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) z[u] = value(p + 64 * u < m ? p + 64 * u : p);
#pragma unroll
        for (int u = 0; u < 4; ++u) k[u] = nearest_level<BITS>(z[u], lv_shared);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (p + 64 * u < m) fit_add<uint64_t>(&acc[k[u]], word(z[u]));
    }
    fit_wave_sync();
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const int k = level_of(i);
        done(i, k < K ? acc[k] : 0);
    }
    fit_wave_sync();
}

}  // namespace qsdp
