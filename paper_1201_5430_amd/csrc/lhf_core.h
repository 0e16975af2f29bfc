// lhf_core.h -- the Gaussian core of the near field (internal).
//
// With u = r^2 / (2 a^2) and S(u) = sum_k (-u)^k / (k! (2k + 3)) the core's factors are
//   f = K / r^3 = sqrt(2/pi) / a^3 S(u),   g = f' / r = sqrt(2/pi) / a^5 S'(u)            (eq. vem1).
// Up to u = 1 both come from polynomials in u.  Beyond, K = 1 - e^-u (erfcx(x) + 2 x / sqrt(pi)), x = sqrt u,
// with erfcx(x) = e^(x^2) erfc(x) as a polynomial in 1 / (x + k), which maps the range to one where it is
// nearly linear; no term cancels there (K >= 0.43).  The polynomials interpolate at Chebyshev nodes in
// 70-digit arithmetic, to relative 1e-18 (S, S') and 4e-18 (erfcx) in FP64, 5e-9 and less in FP32.  With the
// coefficients rounded to the type, as they stand in the tables and enter the sums, evaluated exactly: FP64 S
// 5.7e-17, S' 1.6e-16, erfcx 1.4e-16; FP32 S 1.0e-7, S' 7.2e-8, erfcx 2.0e-7, about a rounding of the type.
// The library's erf and exp with their ranges took most of a pair's time: near field of
// 2^20 uniform elements FP64 1.87 ms with them, 0.94 with these and the lanes split as k_p2p does.
#pragma once

#include <hip/hip_runtime.h>

namespace lhf {
namespace core {

__constant__ double CORE_S64[13] = {
    0.3333333333333333, -0.19999999999999996, 0.0714285714285694, -0.01851851851847368,
    0.0037878787873648332, -0.0006410256375164088, 9.259257719272645e-05, -1.1671289833353212e-05,
    1.305254967800116e-06, -1.3109740748003458e-07, 1.1860014100980693e-08, -9.2647604792917e-10,
    4.875709459963829e-11};
__constant__ double CORE_D64[13] = {
    -0.2, 0.14285714285714282, -0.05555555555555366, 0.01515151515147328, -0.0032051282046482743,
    0.0005555555522785718, -8.16993320241916e-05, 1.0442731233212908e-05, -1.180942296061662e-06,
    1.196949536716896e-07, -1.0909501905328277e-08, 8.572176755184235e-10, -4.529251305805535e-11};
// 1 / k!
__constant__ double EXPM64[14] = {
    1.0, 1.0, 0.5, 1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0, 1.0 / 720.0, 1.0 / 5040.0, 1.0 / 40320.0, 1.0 / 362880.0,
    1.0 / 3628800.0, 1.0 / 39916800.0, 1.0 / 479001600.0, 1.0 / 6227020800.0};
// argument: 11.231433506044905 / (x + 2.5) + -2.208981001727116
__constant__ double ERFCX64[17] = {
    0.20470152155972587, 0.16181313723680746, 0.04866410509652223, 0.010798371077035362,
    0.0015545916565522276, 7.434543328356459e-05, -1.9762478775500553e-05, -3.135980267328544e-06,
    3.219704788340034e-07, 9.22092541150782e-08, -9.369966537798951e-09, -2.7317061956087917e-09,
    4.2474822419831486e-10, 7.367225318873738e-11, -2.1194506302611125e-11, -1.2054228140249565e-12,
    8.423761684691788e-13};
__device__ constexpr double CORE_S32[7] = {
    0.3333333323633967, -0.1999999048334212, 0.07142703950300845, -0.01850921535532344,
    0.0037607273253407497, -0.0005996432911693298, 6.0010976502301616e-05};
__device__ constexpr double CORE_D32[8] = {
    -0.1999999999758284, 0.14285713976063347, -0.055555490256257375, 0.015150988492554666,
    -0.0032030308004320457, 0.0005509789679015834, -7.6071389917114e-05, 6.687078176211976e-06};
// argument: 10.615384615384615 / (x + 2) + -2.5384615384615383
__device__ constexpr double ERFCX32[8] = {
    0.23727272221760473, 0.153218615781747, 0.03285646320681714, 0.004183802453325728,
    0.00010532376631816169, -5.1150929717140246e-05, -3.176206919483035e-06, 9.756948365273017e-07};

// FP32: coefficients as literals of the multiplications
template <int N>
__device__ __forceinline__ float poly(const double (&c)[N], float x)
{
    float r = (float)c[N - 1];
#pragma unroll
    for (int k = N - 2; k >= 0; k--) r = fmaf(r, x, (float)c[k]);
    return r;
}
// FP64: coefficients by scalar loads for each evaluation.  As constants the compiler keeps all of them in
// vector registers over the pair loop (200 of them, two wavefronts per SIMD)
template <int N>
__device__ __forceinline__ double poly64(const double *p, double x)
{
    asm volatile("" : "+s"(p));
    const auto *c = (const __attribute__((address_space(4))) double *)p;
    double r = c[N - 1];
#pragma unroll
    for (int k = N - 2; k >= 0; k--) r = fma(r, x, c[k]);
    return r;
}

// e^-u, 0 <= u <= 46: e^-u = 2^n e^r, |r| <= ln 2 / 2, Taylor's polynomial.  r by Cody and Waite's reduction:
// ln 2 as a first part of 32 bits, whose product with n is exact, and the rest
__device__ __forceinline__ double expm(double u)
{
    const double n = rint(u * -1.4426950408889634074);
    double r = fma(n, -6.93147180369123816490e-01, -u);
    r = fma(n, -1.90821492927058770002e-10, r);
    const double p = poly64<14>(EXPM64, r);
    return ldexp(p, (int)n);
}
// the hardware's 2^t with the rounding of the product t = u log2 e put back
__device__ __forceinline__ float expm(float u)
{
    const float t = u * -1.44269504f;
    const float e = fmaf(u, -1.44269504f, -t) + u * -1.92596299e-8f;
    const float p = __builtin_amdgcn_exp2f(t);
    return fmaf(p, e * 0.693147182f, p);
}
__device__ __forceinline__ double recip(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}
__device__ __forceinline__ float recip(float x)
{
    const float y = __builtin_amdgcn_rcpf(x);
    return fmaf(y, fmaf(-x, y, 1.0f), y);
}
// erfcx(x), 1 <= x <= 6.79 (FP64), 4.9 (FP32)
__device__ __forceinline__ double erfcx(double x)
{
    return poly64<17>(ERFCX64, fma(recip(x + 2.5), 11.231433506044905, -2.208981001727116));
}
__device__ __forceinline__ float erfcx(float x)
{
    return poly(ERFCX32, fmaf(recip(x + 2.0f), 10.615384615384615f, -2.5384615384615383f));
}
__device__ __forceinline__ double sker(double u) { return poly64<13>(CORE_S64, u); }
__device__ __forceinline__ float sker(float u) { return poly(CORE_S32, u); }
__device__ __forceinline__ double dker(double u) { return poly64<13>(CORE_D64, u); }
__device__ __forceinline__ float dker(float u) { return poly(CORE_D32, u); }

}  // namespace core
}  // namespace lhf
