// Functions of a negative score that become its coefficient W = dL/df- and its loss term.  Two forms of each: rows of up to
// KGE_SHORT_SCORES scores take the hardware exp2 / log2 / reciprocal (1 ulp each, about 1e-6 relative: the size of the
// rounding of the fp32 products that the results go into), longer rows the library's functions, whose error does not grow with
// |f|.  Every kernel that forms W from whole rows of scores chooses the same way, when it is launched (LONG): both forms in
// one kernel cost 7 to 15 registers.
#pragma once
#include "kge_common.h"

constexpr int KGE_SHORT_SCORES = 1024;

#ifdef __HIPCC__
namespace {

__device__ __forceinline__ float sigmoidf_(float x) {
    if (x >= 0.f) return 1.f / (1.f + expf(-x));
    const float e = expf(x);
    return e / (1.f + e);
}
__device__ __forceinline__ float softplusf_(float x) { return fmaxf(x, 0.f) + log1pf(expf(-fabsf(x))); }
// Both at once, from one exponential, with the hardware functions
__device__ __forceinline__ void softplus_sigmoid(float f, float& sp, float& sg) {
    const float e = __builtin_amdgcn_exp2f(-fabsf(f) * 1.4426950408889634f);  // exp(-|f|) in (0, 1]
    sp = fmaxf(f, 0.f) + __builtin_amdgcn_logf(1.f + e) * 0.6931471805599453f;
    sg = (f >= 0.f ? 1.f : e) * __builtin_amdgcn_rcpf(1.f + e);
}
template <bool LONG> __device__ __forceinline__ void softplus_sigmoid_of(float f, float& sp, float& sg) {
    if (LONG) {
        sp = softplusf_(f);
        sg = sigmoidf_(f);
    } else {
        softplus_sigmoid(f, sp, sg);
    }
}
// exp of the softmax weights (argument <= 0)
template <bool LONG> __device__ __forceinline__ float softmax_exp(float x) {
    return LONG ? expf(x) : __builtin_amdgcn_exp2f(x * 1.4426950408889634f);
}

}  // namespace
#endif
