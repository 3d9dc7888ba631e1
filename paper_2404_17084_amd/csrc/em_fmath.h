// Elementary functions of the edge terms (device only), FP32 for the mixed path
// and FP64 for the double-precision path.
//
// The FP32 terms are accumulated in FP64 and checked against an FP64 oracle at
// 1e-5 relative per cell, so a few ulp per function are enough; these forms
// replace the correctly rounded library versions, which cost 3-6 times the
// instructions.  Domains are restricted to what the edge terms use.
#pragma once

#include <hip/hip_runtime.h>

namespace em {

// Hardware square root and reciprocal (about 1 ulp).  Arguments of the edge
// terms are 0 or above 2^-100, so no denormal rescaling is needed.
__device__ __forceinline__ float sqrt_f32(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ float rcp_f32(float x) { return __builtin_amdgcn_rcpf(x); }

// atan2(y, x) for y >= 0, result in [0, pi]; (0, 0) gives 0.
// With t = min(|x|, y) / max(|x|, y) in [0, 1], atan t = t P(t^2), P of degree
// 8 fitted for least maximum relative error on [0, 1] (Lawson's iteratively
// reweighted least squares; fit error 1.6e-8), then pi/2 - r when y > |x| and
// pi - r when x < 0.  Within 4 ulp of atan2 with a 1-ulp reciprocal.
__device__ __forceinline__ float atan2_f32(float y, float x)
{
    const float ax = fabsf(x);
    const bool steep = y > ax;  // selects instead of fminf/fmaxf (no NaN handling needed here)
    const float mn = steep ? ax : y, mx = steep ? y : ax;
    const float t = mx > 0.0f ? mn * rcp_f32(mx) : 0.0f;
    const float z = t * t;
    float p = 0.0028501402121037245f;
    p = fmaf(p, z, -0.016069695353507996f);
    p = fmaf(p, z, 0.04269338771700859f);
    p = fmaf(p, z, -0.07504468411207199f);
    p = fmaf(p, z, 0.10641025751829147f);
    p = fmaf(p, z, -0.14203672111034393f);
    p = fmaf(p, z, 0.1999262422323227f);
    p = fmaf(p, z, -0.33333075046539307f);
    p = fmaf(p, z, 1.0f);
    float r = t * p;
    r = steep ? 1.5707963267948966f - r : r;
    return x < 0.0f ? 3.141592653589793f - r : r;
}

// log(1 + u) for u >= 0 (u = 0 gives 0).  1 + u = 2^k m with m in
// [sqrt(1/2), sqrt(2)), f = m - 1 (exact), log m = 2 atanh(s) with
// s = f / (2 + f), |s| <= 0.172, by its series through s^9 (truncation below
// 1e-9 relative).  When 1 + u < 2 the rounding error of 1 + u, u - ((1 + u) - 1),
// is exact and is added back to first order.  Within 5 ulp of log1p with a
// 1-ulp reciprocal.
__device__ __forceinline__ float log1p_f32(float u)
{
    const float v = 1.0f + u;
    int k = __builtin_amdgcn_frexp_expf(v);
    float m = __builtin_amdgcn_frexp_mantf(v);
    if (m < 0.70710678f) {
        m += m;
        k -= 1;
    }
    const float f = m - 1.0f;
    const float s = f * rcp_f32(2.0f + f);
    const float s2 = s * s;
    float p = fmaf(s2, 1.0f / 9.0f, 1.0f / 7.0f);
    p = fmaf(p, s2, 1.0f / 5.0f);
    p = fmaf(p, s2, 1.0f / 3.0f);
    p = fmaf(p, s2, 1.0f);
    const float corr = v < 2.0f ? (u - (v - 1.0f)) * rcp_f32(v) : 0.0f;
    return fmaf((float)k, 0.6931471805599453f, fmaf(s + s, p, corr));
}

// ---------------------------------------------------------------- FP64
// The library's double functions cost several times these (argument classes
// the edge terms never meet, correctly rounded divisions, extended-precision
// intermediate sums).  Each form below is within 3 ulp over its stated domain
// (largest errors found over all exponents and at the cuts: division and square
// root 0.5, arctangent 3.0, logarithm 2.4).

// p z + c with c kept in its register.  The compiler forms the steps of a
// Horner sum as a move of the coefficient and a two-operand v_fmac_f64, one
// instruction more per coefficient than the three-operand form.
__device__ __forceinline__ double horner_f64(double p, double z, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(p), "v"(z), "v"(c));
    return r;
}

// The larger of x and c (fmax quiets its operands by instructions of their own).
__device__ __forceinline__ double max_f64(double x, double c)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(x), "s"(c));
    return r;
}

// n / d for d of ordinary size (no overflow of 1/d): the hardware reciprocal
// (24 bits), one Newton step (48 bits) and a residual correction.
__device__ __forceinline__ double div_f64(double n, double d)
{
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    const double q = n * y;
    return fma(fma(-d, q, n), y, q);
}

// sqrt(x) (0 and infinity are themselves, NaN for NaN and x < 0): the hardware
// reciprocal square root and two coupled Newton steps.
__device__ __forceinline__ double sqrt_f64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return __builtin_amdgcn_class(x, 0x260) ? x : g;  // -0, +0, +infinity
}

// atan2(y, x) for y >= 0, |x| + y < 2^1022; result in [0, pi], (0, 0) gives 0.  Three ranges of
// y / |x|, cut at tan(pi/8) and tan(3 pi/8): the angle is k pi/4 + atan(q) with
// q = y / |x|, (y - |x|) / (y + |x|) or -|x| / y, |q| <= tan(pi/8), one division
// for all three; x < 0 mirrors it to (4 - k) pi/4 - atan(q).  atan q = q + q z
// P(z), z = q^2, P fitted for least maximum relative error (Remez; 4e-17).
__device__ __forceinline__ double atan2_f64(double y, double x)
{
    const double ax = fabs(x);
    const bool low = y <= 0.41421356237309503 * ax, steep = y > 2.4142135623730951 * ax;
    const double num = low ? y : (steep ? -ax : y - ax);
    const double den = max_f64(low ? ax : (steep ? y : y + ax), 0x1p-1022);  // (0, 0): 0 / 2^-1022
    double k = low ? 0.0 : (steep ? 2.0 : 1.0);
    k = x < 0.0 ? 4.0 - k : k;
    const double q = div_f64(x < 0.0 ? -num : num, den), z = q * q;
    double p = 0.021169054961637412741;
    p = horner_f64(p, z, -0.043509553233083249925);
    p = horner_f64(p, z, 0.056894129577670176396);
    p = horner_f64(p, z, -0.06640449782644454278);
    p = horner_f64(p, z, 0.076899799748101054266);
    p = horner_f64(p, z, -0.090907750859824370933);
    p = horner_f64(p, z, 0.11111106273502896402);
    p = horner_f64(p, z, -0.14285714183450741756);
    p = horner_f64(p, z, 0.19999999998888552392);
    p = horner_f64(p, z, -0.33333333333328614107);
    return fma(k, 0.78539816339744831, fma(q * z, p, q));
}

// log(1 + n / d) for n >= 0, d > 0: the ratio of N = d + n and d as 2^k M / D
// with M / D in [5/6, 5/3], log(M / D) = 2 atanh(s), s = (M - D) / (M + D),
// |s| <= 1/4 (n / (2 d + n) when k = 0); atanh s = s + s^3 P(s^2),
// P fitted for least maximum relative error (Remez; 1e-17).  The rounding of N
// is an absolute error where k > 0; with the ratio cut at 5/3 the result is
// above 1/2 there, so that this is one unit (two at a cut of sqrt(2), 3.6 with
// the rest).  One division for the ratio and the logarithm.
__device__ __forceinline__ double log1p_ratio_f64(double n, double d)
{
    const double N = d + n;
    int k = __builtin_amdgcn_frexp_exp(N) - __builtin_amdgcn_frexp_exp(d);
    double M = __builtin_amdgcn_frexp_mant(N), D = __builtin_amdgcn_frexp_mant(d);
    if (M > 1.6666666666666667 * D) {
        D += D;
        k += 1;
    } else if (M < 0.83333333333333337 * D) {
        M += M;
        k -= 1;
    }
    const double s = div_f64(k == 0 ? n : M - D, k == 0 ? fma(2.0, d, n) : M + D), z = s * s;
    double p = 0.07598479913953453;
    p = horner_f64(p, z, 0.06457231710210651);
    p = horner_f64(p, z, 0.07705714463987434);
    p = horner_f64(p, z, 0.09090416066032425);
    p = horner_f64(p, z, 0.11111121626402759);
    p = horner_f64(p, z, 0.14285714161962293);
    p = horner_f64(p, z, 0.2000000000070331);
    p = horner_f64(p, z, 0.33333333333331966);
    const double s2 = s + s;
    return fma((double)k, 0.69314718055994531, fma(s2 * z, p, s2));
}

}  // namespace em
