// Device-side building blocks of the QSDP codec for gfx950 (wave64).
//
// Arithmetic contract (binary32, round to nearest even, no contraction; this file is
// compiled with -ffp-contract=off, fused multiply-adds are written as fmaf):
//   bucket grid   lo = min + 0.0f, hi = max + 0.0f, range = hi - lo,
//                 scale = range / L, inv = L / range (0, 0 for a degenerate bucket: range 0, not
//                 finite, or inv * 2^16 not finite)
//   Q^g           ti = min(trunc(fma(g - lo, inv * 2^16, 1/2)), L * 2^16); code = (ti + h) >> 16, h the
//                 element's 16-bit uniform
//   Q^w (min-max) k = clamp(rint((x - lo) * inv - xi), 0, L); base = fma(xi, scale, lo)
//   Q^w (lattice) k = rint(x / delta - xi); code = min(k - k0, L); base = (k0 + xi) * delta
//   decode        fma(code, scale, base)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qsdp {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11). The key is wave-uniform, so its schedule lives in
// scalar registers; each round costs two 32x32->64 multiplies and two three-operand xors per lane.
// XOR3: an xor of three operands as one v_bitop3_b32 (the compiler makes two v_xor_b32 of it). For the kernels that
// their instructions bind: coin flip onto levels 2 %; the tile kernel's gradient encoder 1-7 % at every width of 2-8
// bits, from fp32 and 16-bit gradients (100M and 60M values, buckets of 96 to 8192; fp32, 8 bits, 8192: 2 % slower);
// the wave kernels' up to 4 bits (128, 1024, 4096: fp32 0-8 %, 16 bits 6-11 %). Above 4 bits these keep the two xors:
// from fp32 the gain is 0-3 % (8 bits 0), from 16-bit gradients it would be 4-9 %. The kernels that memory binds got
// slower with it (fused step over the 1.3B vector 2.53 -> 2.56 ms, code-resident step over 350M 371 -> 382 us).
// ---------------------------------------------------------------------------------------
template <bool XOR3>
__host__ __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    if constexpr (XOR3) return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);  // truth table of a ^ b ^ c
    return a ^ b ^ c;
}

template <bool XOR3 = false>
__host__ __device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4]) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
        const uint32_t n0 = xor3<XOR3>((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n1 = (uint32_t)p1;
        const uint32_t n2 = xor3<XOR3>((uint32_t)(p0 >> 32), c3, k1);
        const uint32_t n3 = (uint32_t)p0;
        c0 = n0; c1 = n1; c2 = n2; c3 = n3;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Rounding uniforms of a row pair: the 16-bit integers h of the lane's eight elements, still packed
// two to a word (low half first). A Philox block (8 elements) spans the lane pair (l even, l+1) of one
// row: the even lane computes the block of the pair's first row, the odd lane that of its second row
// (`block` is the lane's own), and the pair swaps the halves the other needs.
// h[0..1] serve the first row, h[2..3] the second.
template <bool XOR3 = false>
__device__ __forceinline__ void uniforms_of_pair(uint64_t block, int odd, uint32_t k0, uint32_t k1, uint32_t (&h)[4]) {
    uint32_t w[4];
    philox4x32_10<XOR3>((uint32_t)block, (uint32_t)(block >> 32), 0u, 0u, k0, k1, w);
    const uint32_t send0 = odd ? w[0] : w[2];
    const uint32_t send1 = odd ? w[1] : w[3];
    // every lane has a partner, so the destination's previous value never shows
    const uint32_t recv0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)send0, 0xB1, 0xF, 0xF, true);
    const uint32_t recv1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)send1, 0xB1, 0xF, 0xF, true);
    h[0] = odd ? recv0 : w[0]; h[1] = odd ? recv1 : w[1];
    h[2] = odd ? w[2] : recv0; h[3] = odd ? w[3] : recv1;
}

// The same for rows 2c and 2c+1 of a bucket whose lane l holds elements (r*G + l)*4 .. +3 of every row r.
// bucket_block = index of the bucket's first block.
template <int G, bool XOR3 = false>
__device__ __forceinline__ void grad_uniforms_rows(uint64_t bucket_block, int c, int l, uint32_t k0,
                                                   uint32_t k1, uint32_t (&h)[4]) {
    const int odd = l & 1;
    uniforms_of_pair<XOR3>(bucket_block + (uint64_t)(((2 * c + odd) * G + (l - odd)) >> 1), odd, k0, k1, h);
}

// The 16-bit uniform of element i (0..7) of a row pair out of the packed words above.
__device__ __forceinline__ uint32_t uniform16(const uint32_t (&h)[4], int i) {
    return (i & 1) ? (h[i >> 1] >> 16) : (h[i >> 1] & 0xFFFFu);
}

// A shift xi in [-1/2, 1/2): counter 0 of stream 1 (weights) or 2 (shared-shift gradients). Exact in both steps, so the
// host draws the same.
__host__ __device__ __forceinline__ float stream_shift(uint32_t stream, uint32_t k0, uint32_t k1) {
    uint32_t w[4];
    philox4x32_10(0u, 0u, stream, 0u, k0, k1, w);
    return (float)(w[0] >> 8) * 0x1p-24f - 0.5f;
}

// ---------------------------------------------------------------------------------------
// Cross-lane min/max over aligned groups of G lanes (G a power of two, 2..64), all lanes of
// the group end with the result. DPP inside a 16-lane row, gfx950 row/half swaps across rows.
// ---------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    // every lane has a valid source for the controls used here, so the previous value of the
    // destination is irrelevant and the move can fold into the min/max that consumes it
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

__device__ __forceinline__ void swap16(float v, float& a, float& b) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

__device__ __forceinline__ void swap32(float v, float& a, float& b) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

template <int G>
__device__ __forceinline__ float group_min(float v) {
    if (G >= 2) v = fminf(v, dpp_move<0xB1>(v));   // quad_perm [1,0,3,2]
    if (G >= 4) v = fminf(v, dpp_move<0x4E>(v));   // quad_perm [2,3,0,1]
    if (G >= 8) v = fminf(v, dpp_move<0x141>(v));  // row_half_mirror
    if (G >= 16) v = fminf(v, dpp_move<0x140>(v)); // row_mirror
    if (G >= 32) { float a, b; swap16(v, a, b); v = fminf(a, b); }
    if (G >= 64) { float a, b; swap32(v, a, b); v = fminf(a, b); }
    return v;
}

template <int G>
__device__ __forceinline__ float group_max(float v) {
    if (G >= 2) v = fmaxf(v, dpp_move<0xB1>(v));
    if (G >= 4) v = fmaxf(v, dpp_move<0x4E>(v));
    if (G >= 8) v = fmaxf(v, dpp_move<0x141>(v));
    if (G >= 16) v = fmaxf(v, dpp_move<0x140>(v));
    if (G >= 32) { float a, b; swap16(v, a, b); v = fmaxf(a, b); }
    if (G >= 64) { float a, b; swap32(v, a, b); v = fmaxf(a, b); }
    return v;
}

// ---------------------------------------------------------------------------------------
// Per-bucket grids
// ---------------------------------------------------------------------------------------
struct MinMaxGrid {
    float lo, scale, inv;
};

__device__ __forceinline__ MinMaxGrid make_minmax_grid(float lo, float hi, float Lf, bool symmetric) {
    lo = lo + 0.0f;  // -0 -> +0: one bit pattern for the stored base
    hi = hi + 0.0f;
    if (symmetric) {  // grid over [-a, a], a = max |v|
        const float a = fmaxf(fabsf(lo), fabsf(hi));
        lo = -a + 0.0f;
        hi = a;
    }
    const float range = hi - lo;
    const float inv = Lf / range;
    const float scale = range / Lf;
    const bool ok = (range > 0.0f) && (range < __builtin_inff()) && (inv * 65536.0f < __builtin_inff());
    MinMaxGrid g;
    g.lo = lo;
    g.scale = ok ? scale : 0.0f;
    g.inv = ok ? inv : 0.0f;
    return g;
}

// x / delta, as a multiplication when 1/delta is exact (delta a power of two): the product
// and the quotient are then roundings of the same real number.
struct Divider {
    float delta, inv_delta;
    bool pow2;
};

__device__ __forceinline__ float div_delta(float v, const Divider& d) {
    return d.pow2 ? v * d.inv_delta : v / d.delta;
}

// Coin-flip code of one gradient element, decided in integers: the position in the bucket's grid
// in units of 2^-16 of a cell, ti = min(trunc(fma(g - lo, inv * 2^16, 1/2)), L * 2^16) (the
// conversion saturates, so a non-finite input cannot fault), plus the 16-bit uniform h; the code is
// the sum's bits 16 and up: floor(t) + 1 for exactly (ti mod 2^16) of the 2^16 values of h.
__device__ __forceinline__ uint32_t grad_sum16(float g, const MinMaxGrid& grid, uint32_t top16, uint32_t h) {
    const float t16 = fmaf(g - grid.lo, grid.inv * 65536.0f, 0.5f);
    const uint32_t ti = (uint32_t)t16;
    return (ti < top16 ? ti : top16) + h;
}

// ... as a float (for decoding in registers): byte 2 of the sum (the code is at most 255)
__device__ __forceinline__ float grad_code(float g, const MinMaxGrid& grid, uint32_t top16, uint32_t h) {
    return (float)((grad_sum16(g, grid, top16, h) >> 16) & 0xFFu);
}

// ... as an integer (for packing)
__device__ __forceinline__ uint32_t grad_code_int(float g, const MinMaxGrid& grid, uint32_t top16, uint32_t h) {
    return (grad_sum16(g, grid, top16, h) >> 16) & 0xFFu;
}

__device__ __forceinline__ float weight_code_minmax(float x, const MinMaxGrid& grid, float Lf,
                                                    float xi) {
    const float t = (x - grid.lo) * grid.inv;
    const float k = rintf(t - xi);
    return __builtin_amdgcn_fmed3f(k, 0.0f, Lf);
}

// The position of x in the grid before rounding: weight_code_minmax is clamp(rint(this), 0, L).
__device__ __forceinline__ float weight_position_minmax(float x, const MinMaxGrid& grid, float xi) {
    const float t = (x - grid.lo) * grid.inv;
    return t - xi;
}

__device__ __forceinline__ float weight_code_lattice(float x, const Divider& d, float xi, float k0,
                                                     float Lf, uint32_t& saturated) {
    const float k = rintf(div_delta(x, d) - xi);
    float c = k - k0;
    if (c > Lf) {
        c = Lf;
        saturated += 1u;
    }
    return c;
}

// Nearest of K = 2^BITS ascending levels in LDS to z by the plain definition; ties and equal levels resolve to the lowest
// index.
template <int BITS>
__device__ __forceinline__ int nearest_level(float z, const float* lv) {
    constexpr int K = 1 << BITS;
    int j = 0;  // ends as the number of levels < z among the first K-1, i.e. a lower bound
#pragma unroll
    for (int step = K / 2; step >= 1; step >>= 1)
        if (lv[j + step - 1] < z) j += step;
    const int lo_idx = j > 0 ? j - 1 : 0;
    const float d_lo = fabsf(z - lv[lo_idx]);
    const float d_hi = fabsf(z - lv[j]);
    int c = d_hi < d_lo ? j : lo_idx;
    while (c > 0 && lv[c - 1] == lv[c]) --c;  // first among equal levels (rare)
    return c;
}

// ---------------------------------------------------------------------------------------
// Packing: 4 consecutive codes of a lane, 8 consecutive codes (a chunk) = BITS bytes
// ---------------------------------------------------------------------------------------
template <int BITS>
__device__ __forceinline__ uint32_t pack4(const uint32_t (&c)[4]) {
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc |= c[i] << (i * BITS);
    return acc;
}

// Codes given as floats. At 8 bits one instruction per code converts and places it: the conversion to a
// byte rounds to nearest even and saturates to [0, 255], so it also accepts the unrounded grid position
// of weight_position_minmax and then yields clamp(rint(position), 0, 255), the code itself.
template <int BITS>
__device__ __forceinline__ uint32_t pack4(const float (&c)[4]) {
    uint32_t acc = 0;
    if constexpr (BITS == 8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_cvt_pk_u8_f32(c[i], (uint32_t)i, acc);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc |= (uint32_t)c[i] << (i * BITS);
    }
    return acc;
}

// Store the BITS bytes of a packed chunk at byte address p in LDS (p is a multiple of BITS
// bytes from a 16-byte aligned base, so the widest naturally aligned pieces are used).
template <int BITS>
__device__ __forceinline__ void store_chunk(uint8_t* p, uint64_t v) {
    if (BITS == 8) {
        u2 w = {(uint32_t)v, (uint32_t)(v >> 32)};
        *reinterpret_cast<u2*>(p) = w;
    } else if (BITS == 4) {
        *reinterpret_cast<uint32_t*>(p) = (uint32_t)v;
    } else if (BITS == 2) {
        *reinterpret_cast<uint16_t*>(p) = (uint16_t)v;
    } else if (BITS == 6) {
        uint16_t* q = reinterpret_cast<uint16_t*>(p);
        q[0] = (uint16_t)v; q[1] = (uint16_t)(v >> 16); q[2] = (uint16_t)(v >> 32);
    } else {
#pragma unroll
        for (int i = 0; i < BITS; ++i) p[i] = (uint8_t)(v >> (8 * i));
    }
}

template <int BITS>
__device__ __forceinline__ uint64_t load_chunk(const uint8_t* p) {
    if (BITS == 8) {
        u2 w = *reinterpret_cast<const u2*>(p);
        return (uint64_t)w[0] | ((uint64_t)w[1] << 32);
    } else if (BITS == 4) {
        return *reinterpret_cast<const uint32_t*>(p);
    } else if (BITS == 2) {
        return *reinterpret_cast<const uint16_t*>(p);
    } else if (BITS == 6) {
        const uint16_t* q = reinterpret_cast<const uint16_t*>(p);
        return (uint64_t)q[0] | ((uint64_t)q[1] << 16) | ((uint64_t)q[2] << 32);
    } else {
        uint64_t v = 0;
#pragma unroll
        for (int i = 0; i < BITS; ++i) v |= (uint64_t)p[i] << (8 * i);
        return v;
    }
}

// binary32 -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ uint32_t bf16_bits(float v) {
    uint32_t b = __float_as_uint(v);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return b >> 16;
}

// binary32 -> IEEE binary16 bits: the hardware conversion (round to nearest even, subnormal
// results kept, overflow to infinity)
__device__ __forceinline__ uint32_t f16_bits(float v) {
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v);
}

// the 2-byte output formats of the decoders
__device__ __forceinline__ uint32_t half_bits(float v, bool f16) { return f16 ? f16_bits(v) : bf16_bits(v); }

}  // namespace qsdp
