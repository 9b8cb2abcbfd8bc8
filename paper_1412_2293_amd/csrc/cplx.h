// Complex arithmetic shared by the gfx950 kernels of the fused passes.
#pragma once

#include "internal.h"

namespace qs {

template <typename R>
struct cxf {
    R re, im;
};

template <typename R>
__device__ __forceinline__ cxf<R> mul(cxf<R> a, cxf<R> b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}

template <typename R>
__device__ __forceinline__ cxf<R> fma_c(cxf<R> a, cxf<R> b, cxf<R> c)
{
    return {a.re * b.re - a.im * b.im + c.re, a.re * b.im + a.im * b.re + c.im};
}

// A product of many factors that is multiplied into many amplitudes: held with about twice the factors'
// precision (an FP32 product in FP64, an FP64 product as the unevaluated sum hi + lo), because its rounding
// errors are the same for every amplitude it reaches and for every layer with the same factors, and so
// add up where those of single updates average out.
template <typename R>
struct cxprod;

template <>
struct cxprod<float> {
    cxf<double> w;
    __device__ __forceinline__ void clear() { w = {1.0, 0.0}; }
    __device__ __forceinline__ void times(cxf<float> f) { w = mul(w, cxf<double>{f.re, f.im}); }
    __device__ __forceinline__ cxf<float> hi() const { return {(float)w.re, (float)w.im}; }
    __device__ __forceinline__ cxf<float> lo() const
    {
        return {(float)(w.re - (float)w.re), (float)(w.im - (float)w.im)};
    }
};

template <>
struct cxprod<double> {
    cxf<double> h, l;
    __device__ __forceinline__ void clear()
    {
        h = {1.0, 0.0};
        l = {0.0, 0.0};
    }
    // p + q rounded, and what the rounding left out (Knuth's two-sum)
    static __device__ __forceinline__ double sum(double p, double q, double &e)
    {
#pragma clang fp contract(off)
        const double s = p + q, t = s - p;
        e = (p - (s - t)) + (q - t);
        return s;
    }
    // a b + c d rounded, and its error (the products' errors are exact fused multiply-adds)
    static __device__ __forceinline__ double dot(double a, double b, double c, double d, double &e)
    {
#pragma clang fp contract(off)
        const double p = a * b, q = c * d;
        const double s = sum(p, q, e);
        e += __builtin_fma(a, b, -p) + __builtin_fma(c, d, -q);
        return s;
    }
    __device__ __forceinline__ void times(cxf<double> f)
    {
        double er, ei;
        const double re = dot(h.re, f.re, -h.im, f.im, er), im = dot(h.re, f.im, h.im, f.re, ei);
        l = fma_c(l, f, cxf<double>{er, ei});
        h = {re, im};
    }
    __device__ __forceinline__ cxf<double> hi() const { return h; }
    __device__ __forceinline__ cxf<double> lo() const { return l; }
};

// Register-tile element: one complex amplitude as a two-lane vector, so that the compiler keeps
// it in an aligned register pair and moves it with one 64-bit move.
template <typename R>
using tv = R __attribute__((ext_vector_type(2)));
template <typename R>
__device__ __forceinline__ cxf<R> cx(tv<R> v) { return {v.x, v.y}; }
template <typename R>
__device__ __forceinline__ tv<R> tvec(cxf<R> c) { return tv<R>{c.re, c.im}; }
// x times the sum hi + lo
template <typename R>
__device__ __forceinline__ tv<R> mul2(cxf<R> hi, cxf<R> lo, tv<R> x)
{
    return tvec(fma_c(hi, cx<R>(x), mul(lo, cx<R>(x))));
}

// Deposit the low bits of x into the set bits of mask (lowest first).
__device__ __forceinline__ uint32_t deposit32(uint32_t x, uint32_t mask, int K)
{
    uint32_t out = 0;
    int b = 0;
    for (int j = 0; j < K; ++j) {
        if (mask & (1u << j)) {
            out |= ((x >> b) & 1u) << j;
            ++b;
        }
    }
    return out;
}

__device__ __forceinline__ double2 dmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

}  // namespace qs
