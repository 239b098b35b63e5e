// GELU as the linear layers apply it to what they have summed up (internal).
#pragma once

#include "common.h"

namespace ragged {

// GELU(t) = t * Phi(t) = max(t, 0) - |t| * Phi(-|t|), with Phi(-a) = 2^P(a): P has degree 10, P(0) = -1, and keeps the
// RELATIVE error of Phi(-a) small down to the smallest normal fp32 result (a linear program over points of [0, 13.5] whose
// weights are the error bounds below; each bound stands for the whole of its stretch and includes the fp32 evaluation):
//     |t| up to               1     2       3       4       5       7       9       12.9
//     relative error, t < 0   7e-7  1.5e-6  1.7e-5  2.2e-5  1.3e-4  4.2e-3  8.6e-3  3.3e-2
//     relative error, t > 0   5e-7, beyond 1: 1.5e-7
// Nothing cancels in the negative tail.  From about -12.97 on exp2 flushes 2^P < 2^-126, and results below 13 * 2^-126 are 0;
// beyond 13.5 the argument is clamped, so that -infinity gives 0 too.  The maximum is the one that keeps a NaN.
// 13 VALU + 1 transcendental operation per element; the epilogue does not overlap the matrix work, so this count is what the
// activation costs.  (Abramowitz-Stegun 7.1.26 with rcp and exp2, 11 + 2, is further off on every stretch, 24 times from -3 to
// -4.  Degree 6 fitted to the absolute error, 9 + 1, is faster, 25 216 x 3072 x 768 127 against 138 us and 1334 x 3072 x 768
// 11.9 against 12.4, but has no digit left from -9 on and is ten times as far off near 0; degree 9 is up to 1.4 times as far
// off as 7.1.26.)
__device__ __forceinline__ float gelu_erf(float t) {
    const float a = fminf(fabsf(t), 13.5f);
    float p = __builtin_fmaf(a, -2.4868800352351172e-09f, 1.2309047292546893e-07f);
    p = __builtin_fmaf(p, a, -2.41585530602606e-06f);
    p = __builtin_fmaf(p, a, 2.3009282813291065e-05f);
    p = __builtin_fmaf(p, a, -8.495095244143158e-05f);
    p = __builtin_fmaf(p, a, -0.00042139485594816506f);
    p = __builtin_fmaf(p, a, 0.007478408981114626f);
    p = __builtin_fmaf(p, a, -0.052808698266744614f);
    p = __builtin_fmaf(p, a, -0.45909935235977173f);
    p = __builtin_fmaf(p, a, -1.1511178016662598f);
    p = __builtin_fmaf(p, a, -1.0f);
    return __builtin_fmaf(-a, __builtin_amdgcn_exp2f(p), __builtin_elementwise_maximum(t, 0.f));
}

}  // namespace ragged
