// fp32 on the bf16 matrix unit.  The fp32 MFMAs run at a sixteenth of the bf16 rate, and fp32 launches were bound by
// nothing else.  A 24-bit significand is exactly three 8-bit ones with signs of their own: a / 2 = a1 + a2 + a3, a1 the
// nearest bf16 value, a2 the nearest to what that leaves, a3 the rest.  |a2| <= 2^-8 and |a3| <= 2^-17 of a1's binade and of
// either sign, so that the six products a1 b1, a1 b2, a2 b1, a2 b2, a1 b3, a3 b1 leave out at most 2^-24 of a b (half an ulp,
// 2^-27.5 in the root mean square), without a bias; with truncated parts, all of a's sign, it was 2^-21 and 4e-8 towards zero
// on average.  Six bf16 MFMAs take 96 cycles per 16 x 16 x 32 against 256.  (Half of a: rounding the largest values upwards must not
// make them infinite; the products are four times too small until join_parts.  Values below 2^-109 lose their last part.)
//
// The bf16 MFMA truncates what it aligns to a larger sum, so the five small terms have accumulators of their own, added
// to those of a1 b1 at the end: with both in one, sums of positive products fall short by up to 2e-5.
// An infinite or overflowed sum of a1 b1 is the result by itself, since the small parts of an infinity are NaN; a NaN stays one
// in its first part.
#pragma once
#include "common.h"

namespace vgg {

typedef unsigned f32x3_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned f32x3_u32x2 __attribute__((ext_vector_type(2)));

// The parts of half of four values, as bf16 quadruples.
struct Parts4 { f32x3_u32x2 p[3]; };
__device__ __forceinline__ Parts4 split_parts(const f32x3_u32x4 &v)
{
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    // nearest bf16 values of a pair, and what they leave of it
    auto nearest = [](float x, float y) __attribute__((always_inline)) {
        return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2_t{x, y}, bf16x2_t));
    };
    auto low = [](unsigned p) __attribute__((always_inline)) { return __uint_as_float(p << 16); };
    auto high = [](unsigned p) __attribute__((always_inline)) { return __uint_as_float(p & 0xffff0000u); };
    Parts4 o;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float a = __uint_as_float(v[2 * e]), b = __uint_as_float(v[2 * e + 1]);
        const unsigned p = nearest(0.5f * a, 0.5f * b);
        const float ra = __builtin_fmaf(0.5f, a, -low(p)), rb = __builtin_fmaf(0.5f, b, -high(p));
        const unsigned q = nearest(ra, rb);
        o.p[0][e] = p;
        o.p[1][e] = q;
        o.p[2][e] = nearest(ra - low(q), rb - high(q));
    }
    return o;
}

constexpr float kPartsScale = 0.25f;   // of the sums of products of parts
// hi: the sum of a1 b1, lo: that of the smaller terms
__device__ __forceinline__ float join_parts(float hi, float lo) { return (hi + (__builtin_fabsf(hi) < __builtin_inff() ? lo : 0.f)) * (1.f / kPartsScale); }

}  // namespace vgg
