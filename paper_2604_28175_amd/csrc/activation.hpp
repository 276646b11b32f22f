// The activations of the convolution and GEMM kernels' epilogues, in fp32 on the device.
#pragma once
#include "kernels.hpp"

namespace strait {

// GELU: v Phi(v) = max(v, 0) - t q(t) with t = |v| and q(t) = erfc(t / sqrt 2) / 2, the tail of the normal distribution.  log2 q is so smooth that
// a polynomial of degree 8 carries it over 0 .. 6 (least squares, reweighted towards the smallest largest error of t q): the error of the result is at
// most 2.4e-7, 6.7e-8 in the root mean square over -6.5 .. 6.5, and small against the result itself in the negative tail, where fp16 still resolves it
// (relative 5e-4 there, the rounding to fp16).  From t = 6 on t q is below half of fp16's smallest number.  An erf by a rational approximation and exp
// (error 4.6e-7, 1.1e-7; relative 2e-3 in the tail) takes 13 instructions and two of the quarter-rate ones, this 11 and one: the epilogues of the
// feed-forward products are bound by them where a compute unit holds one tile (1024 x 3072 x 768 on 128 x 128 tiles 13.0 -> 12.4 us, 5000 x 3072 x 768 on 256 x 256 tiles 38.0 -> 35.4).
__device__ __forceinline__ float gelu_f(float v) {
    const float t = fminf(fabsf(v), 6.f);
    float p = -3.5990393598694936e-07f;
    p = __builtin_fmaf(p, t, 5.896362381463405e-06f);
    p = __builtin_fmaf(p, t, -4.457409431779524e-06f);
    p = __builtin_fmaf(p, t, -0.0006440711440518498f);
    p = __builtin_fmaf(p, t, 0.007839708589017391f);
    p = __builtin_fmaf(p, t, -0.05313955247402191f);
    p = __builtin_fmaf(p, t, -0.4589434862136841f);
    p = __builtin_fmaf(p, t, -1.1511482000350952f);
    p = __builtin_fmaf(p, t, -0.9999988079071045f);
    return __builtin_fmaf(-t, __builtin_amdgcn_exp2f(p), __builtin_elementwise_maximum(v, 0.f));   // (maximum: a NaN stays one)
}

__device__ __forceinline__ float apply_act(float v, int act) {
    if (act == ACT_RELU) return fmaxf(v, 0.f);
    if (act == ACT_RELU6) return fminf(fmaxf(v, 0.f), 6.f);
    if (act == ACT_GELU) return gelu_f(v);
    return v;
}

}  // namespace strait
