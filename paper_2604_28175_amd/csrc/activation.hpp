// The activations of the convolution and GEMM kernels' epilogues, in fp32 on the device.
#pragma once
#include "kernels.hpp"

namespace strait {

// erf by the rational approximation 7.1.26 of Abramowitz & Stegun (|error| <= 1.5e-7, far below
// the 2^-11 resolution of the fp16 result): 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1/(1 + p|x|).
__device__ __forceinline__ float fast_erf(float x) {
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(1.f + 0.3275911f * ax);
    const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
    const float r = 1.f - poly * __expf(-ax * ax);
    return copysignf(r, x);
}
__device__ __forceinline__ float gelu_f(float v) { return 0.5f * v * (1.f + fast_erf(v * 0.70710678118654752440f)); }

__device__ __forceinline__ float apply_act(float v, int act) {
    if (act == ACT_RELU) return fmaxf(v, 0.f);
    if (act == ACT_RELU6) return fminf(fmaxf(v, 0.f), 6.f);
    if (act == ACT_GELU) return gelu_f(v);
    return v;
}

}  // namespace strait
