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

// Register-tile element: one complex amplitude as a two-lane vector, so that the compiler keeps
// it in an aligned register pair and moves it with one 64-bit move.
template <typename R>
using tv = R __attribute__((ext_vector_type(2)));
template <typename R>
__device__ __forceinline__ cxf<R> cx(tv<R> v) { return {v.x, v.y}; }
template <typename R>
__device__ __forceinline__ tv<R> tvec(cxf<R> c) { return tv<R>{c.re, c.im}; }

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
