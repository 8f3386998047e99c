// fp32 on the bf16 matrix unit.  The fp32 MFMAs run at a sixteenth of the bf16 rate, and fp32 launches were bound by
// nothing else.  A 24-bit significand is exactly three 8-bit ones: a = a1 + a2 + a3, each part the upper half of what the
// parts before it leave (truncated, so that nothing overflows and the parts are exact).  A product takes six bf16 MFMAs,
// all terms down to 2^-24 of it (a1 b1, a1 b2, a2 b1, a2 b2, a1 b3, a3 b1; the three left out are below 2^-27): 96
// cycles per 16 x 16 x 32 against 256.
//
// The bf16 MFMA truncates what it aligns to a larger sum, so the five small terms have accumulators of their own, added
// to those of a1 b1 at the end: with both in one the error grows with a bias (positive operands, 25088 products: 2e-5),
// apart it is a half to a third of the fp32 MFMA's at every length (N(0,1) products, relative 2-norm: 96 terms 0.8e-7
// against 1.8e-7, 1152 2.1e-7 / 6.0e-7, 25088 1.0e-6 / 2.9e-6).  An infinite or overflowed sum of a1 b1 is the result by
// itself, since the small parts of an infinity are NaN.  (Values below 2^-110 lose their last part to underflow.)
#pragma once
#include "common.h"

namespace vgg {

typedef unsigned f32x3_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned f32x3_u32x2 __attribute__((ext_vector_type(2)));

// The parts of four values, as bf16 quadruples.
struct Parts4 { f32x3_u32x2 p[3]; };
__device__ __forceinline__ Parts4 split_parts(const f32x3_u32x4 &v)
{
    unsigned r[4], s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float rest = __uint_as_float(v[e]) - __uint_as_float(v[e] & 0xffff0000u);
        r[e] = __float_as_uint(rest);
        s[e] = __float_as_uint(rest - __uint_as_float(r[e] & 0xffff0000u));
    }
    auto upper = [](unsigned a, unsigned b) __attribute__((always_inline)) { return __builtin_amdgcn_perm(b, a, 0x07060302u); };
    Parts4 o;
    o.p[0] = f32x3_u32x2{upper(v[0], v[1]), upper(v[2], v[3])};
    o.p[1] = f32x3_u32x2{upper(r[0], r[1]), upper(r[2], r[3])};
    o.p[2] = f32x3_u32x2{upper(s[0], s[1]), upper(s[2], s[3])};
    return o;
}

// hi: the sum of a1 b1, lo: that of the smaller terms
__device__ __forceinline__ float join_parts(float hi, float lo) { return hi + (__builtin_fabsf(hi) < __builtin_inff() ? lo : 0.f); }

}  // namespace vgg
