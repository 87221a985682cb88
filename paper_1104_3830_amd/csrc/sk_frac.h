// Exponential of a fraction and logarithm split into integer and fraction, in
// float32 to within about half an ulp, for the kernels that keep a whole
// iteration on chip. The hardware exp2 and log2 are within one ulp each; their
// errors enter every iteration, and a slowly converging instance adds them up
// over its hundreds of iterations.
#pragma once

#include <hip/hip_runtime.h>

namespace sk {

// exp(x) for |x| <= 1/2: the Taylor sum to x^8 (remainder below 6e-9),
// arranged as 1 + (x + x^2 q(x)) so that only the last two additions round at
// the size of the result.
__device__ __forceinline__ float exp_frac(float x) {
    float q = fmaf(x, 1.f / 40320.f, 1.f / 5040.f);
    q = fmaf(q, x, 1.f / 720.f);
    q = fmaf(q, x, 1.f / 120.f);
    q = fmaf(q, x, 1.f / 24.f);
    q = fmaf(q, x, 1.f / 6.f);
    q = fmaf(q, x, 0.5f);
    return 1.f + fmaf(x * x, q, x);
}

__device__ __forceinline__ void exp_frac(float x, float &r) { r = exp_frac(x); }

// The same in float64 to about 3e-10 (terms to x^9), for float64 sums.
__device__ __forceinline__ void exp_frac(float xf, double &r) {
    const double x = xf;
    double q = fma(x, 1.0 / 362880.0, 1.0 / 40320.0);
    q = fma(q, x, 1.0 / 5040.0);
    q = fma(q, x, 1.0 / 720.0);
    q = fma(q, x, 1.0 / 120.0);
    q = fma(q, x, 1.0 / 24.0);
    q = fma(q, x, 1.0 / 6.0);
    q = fma(q, x, 0.5);
    q = fma(q, x, 1.0);
    r = fma(q, x, 1.0);
}

// A potential k + f as it is read: one that a caller split in another way gets
// a fraction, |f| <= 1/2. What neg_log_split and the stage change form stays as
// it is, also where a fraction is past 1/2 by the 1e-4 that neg_log_split
// allows: a potential then has one form, whether it is kept on chip from one
// iteration to the next, read by the next launch or by a caller who resumes
// from it, and no step has to look at it. (Rounding every new potential to
// |f| <= 1/2 instead cost 1 % at n = 64, two dependent instructions a step.)
constexpr float kFracMax = 0.51f;
__device__ __forceinline__ void unit_frac(int &k, float &f) {
    const float r = fabsf(f) > kFracMax ? rintf(f) : 0.f;
    k += (int)r;
    f -= r;
}

// -log(S) = k + f with k an integer, for S in [2^-64, 2^64]; |f| is at most 1/2
// and what the choice of k leaves out (64 kLo and a rounding, under 1e-4).
// S = 2^e m, m in [1/sqrt 2, sqrt 2); with y = m - 1 (exact) and
// s = y / (2 + y), log m = 2 atanh(s) = y - s y + s^3 (2/3 + 2/5 s^2 + ...).
// e log 2 is split so that its leading part and k cancel exactly.
__device__ __forceinline__ float neg_log_split(float S, int &k) {
    float m = __builtin_amdgcn_frexp_mantf(S);  // [1/2, 1)
    int e = __builtin_amdgcn_frexp_expf(S);
    const bool low = m < 0.70710678f;
    m = low ? m + m : m;
    e -= low ? 1 : 0;
    const float y = m - 1.f;
    const float s = y * __builtin_amdgcn_rcpf(2.f + y), z = s * s;
    float r = fmaf(z, 2.f / 11.f, 2.f / 9.f);
    r = fmaf(r, z, 2.f / 7.f);
    r = fmaf(r, z, 2.f / 5.f);
    r = fmaf(r, z, 2.f / 3.f);
    const float corr = s * fmaf(r, z, -y);  // log m = y + corr
    // log 2 = kHi + kLo, kHi a multiple of 2^-15: e kHi is exact
    constexpr float kHi = 22713.f / 32768.f;
    constexpr float kLo = (float)(0.69314718055994530942 - 22713.0 / 32768.0);
    const float ef = (float)e;
    const float gn = -fmaf(ef, kHi, y + corr);
    const float kf = rintf(gn);
    k = (int)kf;
    return (fmaf(-ef, kHi, -kf) - y) - fmaf(ef, kLo, corr);
}

// S in float64: S = T + d with T its float32 rounding, log S = log T + d / T.
__device__ __forceinline__ float neg_log_split(double S, int &k) {
    const float T = (float)S;
    const float d = (float)(S - (double)T);
    return neg_log_split(T, k) - d * __builtin_amdgcn_rcpf(T);
}

}  // namespace sk
