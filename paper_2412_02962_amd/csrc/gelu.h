// Exact-erf GELU of the GEGLU epilogues.
#pragma once

#include "common.h"

namespace pcpp {

// erf by Abramowitz and Stegun, Handbook of Mathematical Functions, formula
// 7.1.26: erf(x) = 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p x) for
// x >= 0, odd extension; absolute error at most 1.5e-7, far below the bf16
// rounding of the products it feeds.
__device__ __forceinline__ float erf_as(float x) {
    const float a = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, a, 1.0f));
    float y = __builtin_fmaf(1.061405429f, t, -1.453152027f);
    y = __builtin_fmaf(y, t, 1.421413741f);
    y = __builtin_fmaf(y, t, -0.284496736f);
    y = __builtin_fmaf(y, t, 0.254829592f);
    y *= t;
    const float e = __builtin_amdgcn_exp2f(-a * a * 1.4426950408889634f);
    return copysignf(__builtin_fmaf(-y, e, 1.0f), x);
}

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erf_as(x * 0.70710678118654752f)); }

}  // namespace pcpp
