// fp32 products on the bf16 matrix cores.
//
// A float is the sum of three bf16 numbers (24 bits of significand in three times 8): x0 = bf16(x), x1 = bf16(x - x0),
// x2 = the rest, |x1| <= 2^-9 |x|, |x2| <= 2^-18 |x|.  That holds from 2^-110 on: the last bits of smaller numbers lie below the
// smallest bf16, 2^-133, and up to 2^-134 is lost (at 1e-34 4.6e-7 of the number).  Of the nine products of two such sums the
// three smallest (2^-27 of the product and less, an eighth of the rounding of one fp32 multiplication) are left out; the other
// six are exact in fp32 and are added up in fp32 by the matrix cores, x0 y0 in one accumulator and the five small ones in
// another.  Six bf16 instructions take 3/8 of the time of the fp32 instructions they replace.  Error against 64 bits, sums of 400
// products of numbers in (-1, 1), relative 2-norm: 0.96e-7, with the fp32 instructions 3.7e-7 (there every product is a rounding
// of the running sum, here sixteen or 32 are added at a time).
#pragma once
#include "kge_common.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// Two floats -> their parts, as pairs of bf16.  Bound by the vector instructions: 11 of them (a conversion of one float
// costs as much as of two).
struct Split2 {
    uint32_t p[3];
};
__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 v;
    v[0] = (__bf16)x;
    v[1] = (__bf16)y;
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float low_bf16(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float high_bf16(uint32_t v) { return __builtin_bit_cast(float, v & 0xffff0000u); }
template <bool LARGE>
__device__ __forceinline__ Split2 split2(float x, float y) {
    // Floats beyond the largest finite bf16 would round to infinity and leave infinity - infinity: they keep it as their first
    // part, and the rest goes into the second.  An infinity is 1, 0 and infinity (with its sign), so that the products of its
    // parts with those of a number, which may have either sign, hold one infinity, that with the number's first part.
    auto first = [](float v) {
        if (!LARGE) return v;
        return __builtin_isinf(v) ? copysignf(1.f, v) : __builtin_amdgcn_fmed3f(v, -3.38953138925e38f, 3.38953138925e38f);
    };
    auto second = [](float v) { return LARGE && __builtin_isinf(v) ? 0.f : v; };
    Split2 s;
    s.p[0] = bf16_pair(first(x), first(y));
    x -= low_bf16(s.p[0]);
    y -= high_bf16(s.p[0]);
    s.p[1] = bf16_pair(second(x), second(y));
    x -= low_bf16(s.p[1]);
    y -= high_bf16(s.p[1]);
    s.p[2] = bf16_pair(x, y);
    return s;
}
// largest magnitude of four floats (NaN: of the others; a NaN needs no clamp, all of its parts are NaN)
__device__ __forceinline__ float magnitude(float4 v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))); }
__device__ __forceinline__ bool is_large(float magnitude) { return magnitude > 3.38953138925e38f; }

struct Split8 {
    bf16x8 p[3];
};

__device__ __forceinline__ void mfma_split(const Split8& a, const Split8& b, floatx4& big, floatx4& small) {
    big = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[0], big, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[1], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[1], b.p[0], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[2], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[2], b.p[0], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[1], b.p[1], small, 0, 0, 0);
}
__device__ __forceinline__ void mfma_split(const Split8& a, const Split8& b, floatx16& big, floatx16& small) {
    big = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[0], b.p[0], big, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[0], b.p[1], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[1], b.p[0], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[0], b.p[2], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[2], b.p[0], small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.p[1], b.p[1], small, 0, 0, 0);
}

}  // namespace
