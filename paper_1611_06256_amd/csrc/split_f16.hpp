// fp32 numbers as two float16 terms, and what scales them.
//
// Scaled by a power of two, x = hi + lo with hi = x rounded to float16 (11 bits) and lo = the rest rounded to float16: 22
// bits and the sign of lo, so that what is left is 2^-23 of x at most, and nothing in three of four numbers of 24 bits.  A
// product of two such numbers is evaluated as lo hi' + hi lo' + hi hi' in the fp32 accumulator of
// v_mfma_f32_16x16x32_f16: three instructions where three bfloat16 terms take six, with two thirds of the operands.  The
// fp32 accumulator rounds half as often, which is what the error of a sum of some hundred products consists of.
//
// The scale brings the largest magnitude of a row or a tensor to [2^14, 2^15).  Numbers below 2^-17 of it are held to 2^-39 of it
// (float16's steps are 2^-24 at least, and the instruction takes such terms as they are).  So a scale is for numbers that go into the same
// sums, and what is contracted against it must not undo its size: filters have one each, a map one as long as its channels are not
// far apart (F16_APART), the operands of weight gradients one for each filter and each channel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "conv1_bf16x3.hpp"

namespace ga3c {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
union F16x8Bits {
    f16x8 v;
    u32x4 u;
};

// Weights too far apart for that: of a filter's weights that are not zero, more than eight or more than one in 32 are below 2^-18 of its
// largest, or that one is no number.  (Where there are few, nothing but small ones may meet an input that is not zero.)  Such a filter's
// reciprocal of the scale is stored as a negative number, and kernels that read it take plain sums instead (conv_plain.hpp).  Of normally
// distributed weights, one in a hundred thousand is that small: nine of a filter's 576, once in 10^26 filters.
constexpr float F16_SMALL = 3.814697265625e-6f;
constexpr int F16_WIDE = 8;
__device__ __forceinline__ bool f16_wide(const int small, const int there) { return small > F16_WIDE || 32 * small > there; }
__device__ __forceinline__ int f16_is_small(const float w, const float most) { return w != 0.f && fabsf(w) < most * F16_SMALL; }

// The power of two by which numbers of magnitude `most` at most are multiplied, and its reciprocal.  Both are normal
// numbers; a tensor of less than 2^-112 stays below 2^14.
__device__ __forceinline__ void f16_scale(const float most, float &scale, float &inverse) {
    const int e = (int)(__float_as_uint(most) >> 23) & 0xff, s = min(268 - e, 253);
    scale = __uint_as_float((uint32_t)s << 23);
    inverse = __uint_as_float((uint32_t)(254 - s) << 23);
}

// Two numbers times `scale` as terms, x in the low halves and y in the high ones: four instructions.
__device__ __forceinline__ void split2_pair(const float x, const float y, const float scale, uint32_t &hi, uint32_t &lo) {
    uint32_t h, l;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(x), "v"(scale));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(y), "v"(scale));
    asm("v_fma_mixlo_f16 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(l) : "v"(x), "v"(scale), "v"(h));
    asm("v_fma_mixhi_f16 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(l) : "v"(y), "v"(scale), "v"(h));
    hi = h;
    lo = l;
}

// The largest of a wavefront's values (none is negative).
__device__ __forceinline__ float f16_wave_most(float m) {
    m = fmaxf(m, dpp_row_f32<0xB1>(m)); m = fmaxf(m, dpp_row_f32<0x4E>(m));
    m = fmaxf(m, dpp_row_f32<0x141>(m)); m = fmaxf(m, dpp_row_f32<0x140>(m));
    const int u = __float_as_int(m);
    return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(u, 0)), __int_as_float(__builtin_amdgcn_readlane(u, 16))),
                 fmaxf(__int_as_float(__builtin_amdgcn_readlane(u, 32)), __int_as_float(__builtin_amdgcn_readlane(u, 48))));
}
// Whether channels of a map, one per lane of a wavefront (some may be there twice), are too far apart for one scale: `size` is what a
// channel's values are of the order of, or at most, the bias of its filter included.  1024: a channel's values are then 2^-10 of the largest ones,
// 2^-18 in a frame of which little is lit, and still good to 2^-21.  (Filters as they are initialised differ by a factor of 1.8 at most; 5000
// updates with a learning rate of 0.1, three hundred times the usual one, made it 19.5, and left no filter with more than one small weight.)
// Channels of zeros don't count.
constexpr float F16_APART = 1024.f;
__device__ __forceinline__ bool f16_apart(const float size) {
    const bool none = size <= 1.1754943508222875e-38f;        // 2^-126: zeros
    return !(f16_wave_most(size) * f16_wave_most(none ? 0.f : 1.f / size) <= F16_APART);        // infinities are apart
}
// The scale of a map whose largest values the eight wavefronts of a block have left in LDS.
__device__ __forceinline__ void f16_scale_of(const float (&m)[8], float &scale, float &inverse) {
    const float a = fmaxf(fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3])), fmaxf(fmaxf(m[4], m[5]), fmaxf(m[6], m[7])));
    f16_scale(__uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(a))), scale, inverse);
}

// ---- Gradients: operands whose magnitude nobody knows before they are there, and sums over several frames.
//
// A scale is its biased exponent here, so that it can be undone in one step (v_ldexp_f32), whatever the two operands' scales are.  What is
// contracted over pixels and frames has one for each row and each column of the product: a filter's dY, a channel's values, so that
// what is far smaller in one filter or channel than in another loses nothing by it.
constexpr int F16_NO_SCALE = 253, F16_ROOM = 2;
__device__ __forceinline__ int f16_exponent(const float most) { return min(268 - (int)(__float_as_uint(most) >> 23 & 0xff), F16_NO_SCALE); }
__device__ __forceinline__ float f16_power(const int exponent) { return __uint_as_float((uint32_t)exponent << 23); }
__device__ __forceinline__ void f16_ldexp4(floatx4 &a, const int4 e, const int more) {
    a[0] = ldexpf(a[0], e.x + more); a[1] = ldexpf(a[1], e.y + more); a[2] = ldexpf(a[2], e.z + more); a[3] = ldexpf(a[3], e.w + more);
}

// ROWS rows of R numbers, one behind the other, that NTHR threads stage: so many neighbouring lanes have a row, four numbers at a time.  The
// last four of a row whose length is no multiple of four overlap the ones before them.
template <int R, int ROWS, int NTHR>
struct F16Rows {
    static constexpr int LANES = NTHR / ROWS, UNITS = (R + 3) / 4, PER = (UNITS + LANES - 1) / LANES;
    static_assert(LANES * ROWS == NTHR && 64 % LANES == 0 && R >= 4, "whole wavefronts of whole rows");
    __device__ static int row(int tid) { return tid / LANES; }
    __device__ static bool there(int tid, int i) { return UNITS % LANES == 0 || tid % LANES + LANES * i < UNITS; }
    __device__ static int at(int tid, int i) { return min(4 * (tid % LANES + LANES * i), R - 4); }           // the first of my numbers in the row
};
// The largest of a row's lanes.
template <int LANES>
__device__ __forceinline__ float f16_row_most(float m) {
    if constexpr (LANES == 64) return f16_wave_most(m);
    if constexpr (LANES >= 2) m = fmaxf(m, dpp_row_f32<0xB1>(m));
    if constexpr (LANES >= 4) m = fmaxf(m, dpp_row_f32<0x4E>(m));
    if constexpr (LANES >= 8) m = fmaxf(m, dpp_row_f32<0x141>(m));
    if constexpr (LANES >= 16) m = fmaxf(m, dpp_row_f32<0x140>(m));
    if constexpr (LANES >= 32) m = fmaxf(m, __shfl_xor(m, 16));
    return m;
}
// The exponent of my row's scale, which has been `e`: where that is too large for what all(fold) folds, one that leaves room for four
// times as much, so that few frames change it.  Infinities don't count (in a second look, which only they cost), NaN never do.
template <int LANES, class All>
__device__ __forceinline__ int f16_row_exponent(const int e, const All &all) {
    float m = 0.f;
    all([&](const float v) { m = fmaxf(m, fabsf(v)); });
    m = f16_row_most<LANES>(m);
    if (__any(m == __builtin_inff())) {
        m = 0.f;
        all([&](const float v) { const float a = fabsf(v); m = fmaxf(m, a < __builtin_inff() ? a : 0.f); });
        m = f16_row_most<LANES>(m);
    }
    const int need = f16_exponent(m);
    return need < e ? need - F16_ROOM : e;
}

// One of the operands' terms times the other's: bfloat16 (one term) or float16.
template <bool BF16>
__device__ __forceinline__ floatx4 mfma_terms(const u32x4 a, const u32x4 b, const floatx4 c) {
    if constexpr (BF16) {
        Bf16x8Bits x, y;
        x.u = a; y.u = b;
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.v, y.v, c, 0, 0, 0);
    } else {
        F16x8Bits x, y;
        x.u = a; y.u = b;
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(x.v, y.v, c, 0, 0, 0);
    }
}
// Three products a sum, smallest first, or the one of rounded operands.
template <bool ONE> constexpr int F16_PRODUCTS = ONE ? 1 : 3;
template <bool ONE> constexpr int f16_a_term(int q) { return ONE ? 0 : q == 0; }
template <bool ONE> constexpr int f16_b_term(int q) { return ONE ? 0 : q == 1; }

// Two values as terms: bfloat16, rounded (the others are not used), or two of float16.
template <bool ONE>
__device__ __forceinline__ void split_terms(const float x, const float y, const float scale, uint32_t (&t)[2]) {
    if constexpr (ONE) {
        uint32_t mid, lo;
        split3_pair(x, y, t[0], mid, lo);
        t[1] = 0;
    } else {
        split2_pair(x, y, scale, t[0], t[1]);
    }
}

// Two bytes, in the low halves of a register's halves under 0x64, as float16: 1024 + b is 0x6400 | b.  (A byte's bits alone are those of the
// subnormal number b 2^-24, which the matrix instruction takes as if it were 2^-14: bits of the running sum that are small against
// that are dropped, and sums of dark frames were 3e-5 off.)
__device__ __forceinline__ uint32_t f16_pair_of_bytes(const uint32_t b) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    union { uint32_t u; f16x2 v; } c;
    c.u = b;
    c.v -= f16x2{1024.f, 1024.f};
    return c.u;
}
// Eight bytes.
__device__ __forceinline__ f16x8 f16_of_bytes(const uint32_t lo, const uint32_t hi) {
    constexpr uint32_t UP = 0x64646464u;
    F16x8Bits v;
    v.u = u32x4{f16_pair_of_bytes(__builtin_amdgcn_perm(UP, lo, 0x04010400u)), f16_pair_of_bytes(__builtin_amdgcn_perm(UP, lo, 0x04030402u)),
                f16_pair_of_bytes(__builtin_amdgcn_perm(UP, hi, 0x04010400u)), f16_pair_of_bytes(__builtin_amdgcn_perm(UP, hi, 0x04030402u))};
    return v.v;
}

// A frame of 4 x 84 x 84 bytes in LDS, as it lies in memory, where it comes without passing through registers; NW wavefronts, 16
// bytes per lane and load.  The last load's lanes behind the frame's end fill the place up with its last bytes.
constexpr int F16_FRAME = 28 * 1024;
template <int NW>
__device__ __forceinline__ void f16_frame_to_lds(const uint8_t *src, const uint32_t lds, const int wave, const int lane) {
    constexpr int LAST = 4 * 84 * 84 / 1024, REST = (4 * 84 * 84 % 1024) / 16;
#pragma unroll
    for (int i = 0; i < (LAST + NW) / NW; ++i) {
        const int p = wave + NW * i;
        if (p < LAST) load_vec_to_lds(src + 1024 * p, 16u * lane, lds + 1024 * p);
        else if (p == LAST) load_vec_to_lds(src + 1024 * p, 16u * min(lane, REST - 1), lds + 1024 * p);
    }
}

}  // namespace ga3c
