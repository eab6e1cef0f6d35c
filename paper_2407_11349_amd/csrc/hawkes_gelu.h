// hawkes_gelu.h -- GELU x Phi(x) and its derivatives in FP32 (device code of the
// surrogate network).
#ifndef HAWKES_GELU_H
#define HAWKES_GELU_H

#include <hip/hip_runtime.h>

namespace hawkes {

constexpr float K_SQRT1_2 = 0.70710678118654752440f;
constexpr float K_INV_SQRT_2PI = 0.39894228040143267794f;

__device__ inline float gelu(float x) { return 0.5f * x * (1.0f + erff(x * K_SQRT1_2)); }
__device__ inline float gelu_d1(float x)
{
    return 0.5f * (1.0f + erff(x * K_SQRT1_2)) + x * K_INV_SQRT_2PI * expf(-0.5f * x * x);
}
__device__ inline float gelu_d2(float x) { return K_INV_SQRT_2PI * expf(-0.5f * x * x) * (2.0f - x * x); }

// GELU and its slope Phi + x phi from one exponential, for batched inference (training
// keeps erff and expf): Phi(-u) = e R with e = exp(-u^2/2), u = |x|, where R (half the scaled
// complementary error function at u/sqrt 2) is a degree-7 polynomial in w = u / (u + 4), 1/2 at
// w = 0, with the least largest error of u Phi(-u) and Phi(-u) over 0 <= u <= 13.5, 1.2e-8
// (Lawson's iteration, the coefficients rounded one after the other; of the shifts 3.2 to 4.3 and degrees 7
// and 8, the shortest at that error).  w is small where R is steep, so the reciprocal's rounding does not count
// there, and each result ends in one fma: GELU x/2 + |x| (1/2 - e R), slope
// e (R - u / sqrt(2 pi)) for x < 0 and one minus that above.  w is held within [0, 1] (by its product's clamp), so
// that an infinite x gives what erff gives.
//   Errors (largest, rms) over 2^22 standard normal x: GELU 2.7e-7, 2.0e-8 and slope 1.0e-7,
// 2.3e-8; with erff and expf 3.9e-7, 2.5e-8 and 1.4e-7, 2.7e-8; with a polynomial in 1 / (1 + 0.27 u) and the slope
// added to a rounded Phi 3.6e-7, 2.5e-8 and 2.4e-7, 4.2e-8 (in the same time: 38.7 us for 21,000
// samples, 526 for 400,000).  Some 22 instructions instead of 75, which were the kernel's largest part by far.
struct Gelu {
    float a, d1;
};
__device__ __forceinline__ Gelu gelu_all(float x)
{
    const float u = fabsf(x);
    const float w = fminf(fmaxf(u * __builtin_amdgcn_rcpf(u + 4.0f), 0.0f), 1.0f);
    const float e = __builtin_amdgcn_exp2f(x * x * -0.72134752044448170368f);
    float r = 9.630157799e-02f;
    r = fmaf(r, w, -3.094779551e-01f);
    r = fmaf(r, w, 1.486228257e-01f);
    r = fmaf(r, w, 8.615880013e-01f);
    r = fmaf(r, w, -2.105239391e+00f);
    r = fmaf(r, w, 2.404155731e+00f);
    r = fmaf(r, w, -1.595767736e+00f);
    r = fmaf(r, w, 0.5f);
    const float k = fmaf(-K_INV_SQRT_2PI, u, r);
    const bool p = x >= 0.0f;
    return Gelu{fmaf(fabsf(x), fmaf(-r, e, 0.5f), 0.5f * x), fmaf(p ? -e : e, k, p ? 1.0f : 0.0f)};
}

}  // namespace hawkes

#endif  // HAWKES_GELU_H
