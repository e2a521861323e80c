// Accumulation of the layer recurrence on the device: complex types, the plain
// complex multiply-add and the compensated complex64 accumulators, shared by
// the tiled layer kernel (layer.hip) and the table-driven ones (flat.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "slos_internal.h"

namespace {

template <typename T> struct Cx;
template <> struct Cx<float> { using type = float2; };
template <> struct Cx<double> { using type = double2; };

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// acc += u * v (complex), four fused multiply-adds
template <typename C>
__device__ __forceinline__ void cmac(C &acc, const C u, const C v)
{
    acc.x = fma_(u.x, v.x, acc.x);
    acc.x = fma_(-u.y, v.y, acc.x);
    acc.y = fma_(u.x, v.y, acc.y);
    acc.y = fma_(u.y, v.x, acc.y);
}

// |a|^2 with one rounding order in every kernel (left to the compiler, either
// product may be the fused one)
__device__ __forceinline__ double prob(double re, double im) { return __builtin_fma(re, re, im * im); }

// ---- compensated complex64 accumulation ---------------------------------
// SLOS_COMP_TWOSUM: every real product a*b is split exactly into p + pe with an
// FMA (two-product) and added to the running sum s with Knuth's two-sum; both
// rounding errors go to a second float c.  Ten operations per product.
__device__ __forceinline__ void acc_exact(float &s, float &c, float a, float b)
{
#pragma clang fp contract(off)
    float p = a * b;
    float pe = __builtin_fmaf(a, b, -p);
    float t = s + p;
    float bb = t - s;
    float e = (s - (t - bb)) + (p - bb);
    s = t;
    c = c + (e + pe);
}

struct CompAcc {
    float2 s, c;
};

__device__ __forceinline__ void cmac_comp(CompAcc &a, const float2 u, const float2 v)
{
    acc_exact(a.s.x, a.c.x, u.x, v.x);
    acc_exact(a.s.x, a.c.x, -u.y, v.y);
    acc_exact(a.s.y, a.c.y, u.x, v.y);
    acc_exact(a.s.y, a.c.y, u.y, v.x);
}

// Default compensated mode: biased FMA accumulation.  The sum starts at a
// power of two sigma >= 4 * sum_i |a_i b_i| (a bound known before the sum).  Every partial sum then stays within [3/4, 5/4] sigma, so
// for t = fma(a, b, s) the difference s - t is exact (Sterbenz) and
// fma(a, b, s - t) is the FMA's rounding error, correct to one rounding of a
// number below ulp(sigma).  Those errors go to a second float c, and the
// result is (s - sigma) + c, where s - sigma is exact again.  The error-free
// transformation is the two-sum of s and a*b computed with the FMA; the bias
// makes its short form exact.  Four operations per real product; the error is
// within one rounding of the result plus O(terms * 2^-46 * sigma).
__device__ __forceinline__ void acc_biased(float &s, float &c, float a, float b)
{
#pragma clang fp contract(off)
    const float t = __builtin_fmaf(a, b, s);
    const float d = s - t;
    c = c + __builtin_fmaf(a, b, d);
    s = t;
}

// 8 * 2^floor(log2 b) (> 4b), at least 2^-117
__device__ __forceinline__ float bias_for(float b)
{
    const float f = __uint_as_float(__float_as_uint(b) & 0x7F800000u);
    return 8.0f * fmaxf(f, 0x1p-120f);
}

template <typename T, int COMP> struct Acc;
template <typename T> struct Acc<T, SLOS_COMP_NONE> {
    using C = typename Cx<T>::type;
    C a;
    __device__ __forceinline__ void zero() { a = C{0, 0}; }
    __device__ __forceinline__ void start(float) {}
    __device__ __forceinline__ void mac(const C u, const C v) { cmac(a, u, v); }
    __device__ __forceinline__ C value() const { return a; }
    __device__ __forceinline__ double re() const { return (double)a.x; }
    __device__ __forceinline__ double im() const { return (double)a.y; }
};
template <> struct Acc<float, SLOS_COMP_TWOSUM> {
    CompAcc a;
    __device__ __forceinline__ void zero() { a.s = float2{0.f, 0.f}; a.c = float2{-0.f, -0.f}; }
    __device__ __forceinline__ void start(float) {}
    __device__ __forceinline__ void mac(const float2 u, const float2 v) { cmac_comp(a, u, v); }
    __device__ __forceinline__ float2 value() const { return float2{a.s.x + a.c.x, a.s.y + a.c.y}; }
    __device__ __forceinline__ double re() const { return (double)a.s.x + (double)a.c.x; }
    __device__ __forceinline__ double im() const { return (double)a.s.y + (double)a.c.y; }
};
template <> struct Acc<float, SLOS_COMP_BIASED> {
    float sr, si, cr, ci, sigma;
    // the error sums start at -0, the identity of IEEE addition, so the first
    // term's addition folds away
    __device__ __forceinline__ void zero()
    {
        sr = si = sigma = 0.f;
        cr = ci = -0.f;
    }
    __device__ __forceinline__ void start(float bias)
    {
        sigma = bias;
        sr = bias;
        si = bias;
    }
    __device__ __forceinline__ void mac(const float2 u, const float2 v)
    {
        acc_biased(sr, cr, u.x, v.x);
        acc_biased(sr, cr, -u.y, v.y);
        acc_biased(si, ci, u.x, v.y);
        acc_biased(si, ci, u.y, v.x);
    }
    __device__ __forceinline__ float2 value() const { return float2{(sr - sigma) + cr, (si - sigma) + ci}; }
    __device__ __forceinline__ double re() const { return (double)(sr - sigma) + (double)cr; }
    __device__ __forceinline__ double im() const { return (double)(si - sigma) + (double)ci; }
};

// FP64 mode: each term's complex64 factors are widened to FP64, where their
// products are exact (24-bit significands), and the products are summed with
// FP64 FMAs: one FP64 rounding per real product, four FMAs and up to four
// conversions per complex term (the FP64 FMA issues at the FP32 rate here).
template <> struct Acc<float, SLOS_COMP_F64> {
    double r, i;
    __device__ __forceinline__ void zero() { r = i = 0.0; }
    __device__ __forceinline__ void start(float) {}
    __device__ __forceinline__ void mac(const float2 uf, const float2 v)
    {
        const double2 u{(double)uf.x, (double)uf.y};
        const double vr = (double)v.x, vi = (double)v.y;
        r = __builtin_fma(u.x, vr, r);
        r = __builtin_fma(-u.y, vi, r);
        i = __builtin_fma(u.x, vi, i);
        i = __builtin_fma(u.y, vr, i);
    }
    __device__ __forceinline__ float2 value() const { return float2{(float)r, (float)i}; }
    __device__ __forceinline__ double re() const { return r; }
    __device__ __forceinline__ double im() const { return i; }
};

} // namespace
