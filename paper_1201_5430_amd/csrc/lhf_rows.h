// lhf_rows.h -- what the kernels with a vector split over the four 16-lane rows of a wavefront share
// (internal): multiplication by an entry broadcast within the row, and swaps of rows.
#pragma once

#include <hip/hip_runtime.h>

namespace lhf {
namespace tr {

// a += (entry K of the row's 16 w) x
template <int K>
__device__ __attribute__((always_inline)) inline void fmab(double &a, double w, double x)
{
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(a) : "v"(w), "v"(x), "n"(K));
}
template <int K>
__device__ __attribute__((always_inline)) inline void fmab(float &a, float w, float x)
{
    asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(a) : "v"(w), "v"(x), "n"(K));
}

// (a, b) -> (a of the even rows | b of the even rows, a of the odd rows | b of the odd rows); X = 32: of
// the lower and the upper half
template <int X>
__device__ __attribute__((always_inline)) inline void swap1(unsigned &a, unsigned &b)
{
    if constexpr (X == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    }
}
template <int X>
__device__ __attribute__((always_inline)) inline void swap(float &a, float &b)
{
    unsigned u = __float_as_uint(a), v = __float_as_uint(b);
    swap1<X>(u, v);
    a = __uint_as_float(u);
    b = __uint_as_float(v);
}
template <int X>
__device__ __attribute__((always_inline)) inline void swap(double &a, double &b)
{
    const unsigned long long p = __double_as_longlong(a), q = __double_as_longlong(b);
    unsigned pl = (unsigned)p, ph = (unsigned)(p >> 32), ql = (unsigned)q, qh = (unsigned)(q >> 32);
    swap1<X>(pl, ql);
    swap1<X>(ph, qh);
    a = __longlong_as_double((long long)(((unsigned long long)ph << 32) | pl));
    b = __longlong_as_double((long long)(((unsigned long long)qh << 32) | ql));
}
__device__ __attribute__((always_inline)) inline float flip(float x, unsigned s)
{
    return __uint_as_float(__float_as_uint(x) ^ s);
}
__device__ __attribute__((always_inline)) inline double flip(double x, unsigned s)
{
    return __longlong_as_double(__double_as_longlong(x) ^ (long long)((unsigned long long)s << 32));
}

}  // namespace tr

}  // namespace lhf
