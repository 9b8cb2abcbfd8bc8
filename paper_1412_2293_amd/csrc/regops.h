// Gate updates of a thread's register tile (the amplitude-pair update of Section 2 and its
// two-qubit form), shared by the kernels that run register rounds.
#pragma once

#include "cplx.h"

namespace qs {

// Phase factors of one folded block for this thread: w (tile and thread constant) and one
// factor per register bit, applied to a pair when that bit of the pair index is 1.
template <typename R, int RB>
struct PhaseSet {
    cxf<R> w;
    cxf<R> bit[RB];
    bool any;
};

// grec: the block in global memory (uniform reads, held in scalar registers); lrec: the same
// block staged in LDS (per-thread table lookups); wout: this tile's products of the phases
// conditioned on tile-number bits (global memory, uniform reads).
// bits: whether the block has phases conditioned on register bits (else only w is used).
// uni: no factor of the block depends on a thread-id bit, so every entry of the thread tables
// equals their first (uniform reads instead of per-thread lookups).
template <typename R, int RB>
__device__ __forceinline__ void load_phases(PhaseSet<R, RB> &ps, const cxf<R> *__restrict__ grec,
                                            const cxf<R> *lrec, bool present, bool bits, bool uni, int job,
                                            const cxf<R> *wout, uint32_t tid)
{
    ps.any = present;
    if (!present) return;
    if (bits) {
#pragma unroll
        for (int k = 0; k < RB; ++k) ps.bit[k] = grec[k];
    }
    if (uni) ps.w = grec[4];
    else ps.w = mul(lrec[4 + (tid & 31u)], lrec[36 + ((tid >> 5) & 15u)]);
    if (job >= 0) ps.w = mul(ps.w, wout[job]);
}

// Phase of the pair at register index r: w, times the register-bit factors when BITS.
template <typename R, int RB, int P, bool BITS>
__device__ __forceinline__ cxf<R> pair_phase(const PhaseSet<R, RB> &ps, int r)
{
    cxf<R> w = ps.w;
    if constexpr (BITS) {
#pragma unroll
        for (int q = 0; q < RB; ++q)
            if (q != P && ((r >> q) & 1)) w = mul(w, ps.bit[q]);
    }
    return w;
}

// Register index of the k-th pair (bit P clear) and of the k-th quadruple (bits P0, P1 clear):
// compile-time integer arithmetic, so that after unrolling every register access is static.
template <int P>
__device__ constexpr int pair_base(int k)
{
    return ((k >> P) << (P + 1)) | (k & ((1 << P) - 1));
}

template <int P0, int P1>
__device__ constexpr int quad_base(int k)
{
    constexpr int lo = P0 < P1 ? P0 : P1, hi = P0 < P1 ? P1 : P0;
    return pair_base<hi>(pair_base<lo>(k));
}

// PRE: input phase kind (0 none, 1 one factor per thread, 2 with register-bit factors); POST:
// the folded output block (0 none, 1 one factor per thread, 2 with register-bit factors; with
// one factor it joins the |1> row of the matrix once per op instead of a product per pair).  ZIN: which input of every pair is known to be
// zero (0 neither; 1 the |1> input, 2 the |0> input) -- the target qubit has not been touched by
// any earlier gate of the run and still holds the basis bit 0 (1), so that half of the tile is
// exactly zero and its products are left out (the result is the same: a product with zero
// added to a value leaves the value).  They are uniform per op, so each combination is its own
// straight-line code behind a scalar branch, with no work for an absent block.
template <typename R, int RB, int P, int PRE, int POST, int ZIN>
__device__ __forceinline__ void apply_u1(tv<R> (&a)[1 << RB], const cxf<R> (&m0)[4],
                                         const PhaseSet<R, RB> &pre, const PhaseSet<R, RB> &post)
{
    cxf<R> m[4] = {m0[0], m0[1], m0[2], m0[3]};
    if constexpr (POST == 1) {
        m[2] = mul(post.w, m[2]);
        m[3] = mul(post.w, m[3]);
    }
#pragma unroll
    for (int k = 0; k < (1 << (RB - 1)); ++k) {
        const int r = pair_base<P>(k);
        const int r1 = r | (1 << P);
        cxf<R> x0 = cx<R>(a[r]), x1 = cx<R>(a[r1]);
        cxf<R> y0, y1;
        if constexpr (ZIN == 1) {
            y0 = mul(m[0], x0);
            y1 = mul(m[2], x0);
        } else {
            if constexpr (PRE > 0) x1 = mul(pair_phase<R, RB, P, PRE == 2>(pre, r), x1);
            if constexpr (ZIN == 2) {
                y0 = mul(m[1], x1);
                y1 = mul(m[3], x1);
            } else {
                y0 = fma_c(m[1], x1, mul(m[0], x0));
                y1 = fma_c(m[3], x1, mul(m[2], x0));
            }
        }
        if constexpr (POST == 2) y1 = mul(pair_phase<R, RB, P, true>(post, r), y1);
        a[r] = tvec(y0);
        a[r1] = tvec(y1);
    }
}

// The same update with a real matrix (m[k].im == 0): half the multiplications.  A one-factor
// output block makes the |1> row complex (m2 w, m3 w).
template <typename R, int RB, int P, int PRE, int POST, int ZIN>
__device__ __forceinline__ void apply_u1_real(tv<R> (&a)[1 << RB], const cxf<R> (&m)[4],
                                              const PhaseSet<R, RB> &pre, const PhaseSet<R, RB> &post)
{
    const R m0 = m[0].re, m1 = m[1].re, m2 = m[2].re, m3 = m[3].re;
    cxf<R> m2w, m3w;
    if constexpr (POST == 1) {
        m2w = {m2 * post.w.re, m2 * post.w.im};
        m3w = {m3 * post.w.re, m3 * post.w.im};
    }
#pragma unroll
    for (int k = 0; k < (1 << (RB - 1)); ++k) {
        const int r = pair_base<P>(k);
        const int r1 = r | (1 << P);
        cxf<R> x0 = cx<R>(a[r]), x1 = cx<R>(a[r1]);
        cxf<R> y0, y1;
        if constexpr (ZIN == 1) {
            y0 = {m0 * x0.re, m0 * x0.im};
            if constexpr (POST == 1) y1 = mul(m2w, x0);
            else y1 = {m2 * x0.re, m2 * x0.im};
        } else {
            if constexpr (PRE > 0) x1 = mul(pair_phase<R, RB, P, PRE == 2>(pre, r), x1);
            if constexpr (ZIN == 2) {
                y0 = {m1 * x1.re, m1 * x1.im};
                if constexpr (POST == 1) y1 = mul(m3w, x1);
                else y1 = {m3 * x1.re, m3 * x1.im};
            } else {
                y0 = {m0 * x0.re + m1 * x1.re, m0 * x0.im + m1 * x1.im};
                if constexpr (POST == 1) y1 = fma_c(m3w, x1, mul(m2w, x0));
                else y1 = {m2 * x0.re + m3 * x1.re, m2 * x0.im + m3 * x1.im};
            }
        }
        if constexpr (POST == 2) y1 = mul(pair_phase<R, RB, P, true>(post, r), y1);
        a[r] = tvec(y0);
        a[r1] = tvec(y1);
    }
}

// The update of a sheared reflection (OPF_SHEAR), up to its factor alpha: two multiply-adds per pair
// and component, each rounded once, instead of four operations (Grover n = 20, complex<float>, 64
// trajectories, 16 iterations: 7.65 ms a run, 9.37 with the matrices; the passes are bound by issue).
template <typename R, int RB, int P>
__device__ __forceinline__ void apply_u1_shear(tv<R> (&a)[1 << RB], R t)
{
#pragma unroll
    for (int k = 0; k < (1 << (RB - 1)); ++k) {
        const int r = pair_base<P>(k), r1 = r | (1 << P);
        const tv<R> x0 = a[r], x1 = a[r1];
        a[r] = tv<R>{__builtin_elementwise_fma(t, x1.x, x0.x), __builtin_elementwise_fma(t, x1.y, x0.y)};
        a[r1] = tv<R>{__builtin_elementwise_fma(t, x0.x, -x1.x), __builtin_elementwise_fma(t, x0.y, -x1.y)};
    }
}

template <typename R, int RB>
__device__ __forceinline__ void dispatch_u1_shear(int p, tv<R> (&a)[1 << RB], R t)
{
    if (RB > 1 && p == 0) apply_u1_shear<R, RB, 0>(a, t);
    else if (RB > 2 && p == 1) apply_u1_shear<R, RB, 1 % RB>(a, t);
    else if (RB > 3 && p == 2) apply_u1_shear<R, RB, 2 % RB>(a, t);
    else apply_u1_shear<R, RB, RB - 1>(a, t);
}

// A one-qubit update on a target that still holds its basis bit, with a real matrix and one
// uniform output factor: one input of every pair is exactly zero (which one is the basis bit),
// so their sum is the other; the |0> output is A times it (A real), the |1> output B times it.
template <typename R, int RB, int P>
__device__ __forceinline__ void apply_u1_untouched(tv<R> (&a)[1 << RB], R A, cxf<R> B)
{
#pragma unroll
    for (int k = 0; k < (1 << (RB - 1)); ++k) {
        const int r = pair_base<P>(k);
        const int r1 = r | (1 << P);
        const cxf<R> x = {a[r].x + a[r1].x, a[r].y + a[r1].y};
        a[r] = tv<R>{A * x.re, A * x.im};
        a[r1] = tvec(mul(B, x));
    }
}

// REAL: the 4 x 4 matrix is real (a permutation, or the superoperator of a real Kraus set on
// vec(rho)): two multiply-adds per product instead of four.
template <typename R, int RB, int P0, int P1, bool REAL>
__device__ __forceinline__ void apply_u2(tv<R> (&a)[1 << RB], const cxf<R> (&m)[16])
{
#pragma unroll
    for (int k = 0; k < (1 << (RB - 2)); ++k) {
        const int r0 = quad_base<P0, P1>(k);
        const int r1 = r0 | (1 << P0), r2 = r0 | (1 << P1), r3 = r0 | (1 << P0) | (1 << P1);
        const cxf<R> x0 = cx<R>(a[r0]), x1 = cx<R>(a[r1]), x2 = cx<R>(a[r2]), x3 = cx<R>(a[r3]);
        cxf<R> y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (REAL) {
                const R c0 = m[4 * i].re, c1 = m[4 * i + 1].re, c2 = m[4 * i + 2].re, c3 = m[4 * i + 3].re;
                y[i] = {c0 * x0.re + c1 * x1.re + c2 * x2.re + c3 * x3.re,
                        c0 * x0.im + c1 * x1.im + c2 * x2.im + c3 * x3.im};
            } else {
                cxf<R> s = mul(m[4 * i], x0);
                s = fma_c(m[4 * i + 1], x1, s);
                s = fma_c(m[4 * i + 2], x2, s);
                s = fma_c(m[4 * i + 3], x3, s);
                y[i] = s;
            }
        }
        a[r0] = tvec(y[0]);
        a[r1] = tvec(y[1]);
        a[r2] = tvec(y[2]);
        a[r3] = tvec(y[3]);
    }
}

// Dispatch on the target register bit.  There is no pass-through branch (the last position
// is the fall-back): every path rewrites the register tile, which lets the register allocator
// keep the tile in the same registers across ops instead of copying it at each merge.
template <typename R, int RB, int PRE, int POST, int ZIN>
__device__ __forceinline__ void dispatch_u1_pp(int p, bool real, tv<R> (&a)[1 << RB], const cxf<R> (&m)[4],
                                               const PhaseSet<R, RB> &pre, const PhaseSet<R, RB> &post)
{
    if (real) {
        if (RB > 1 && p == 0) apply_u1_real<R, RB, 0, PRE, POST, ZIN>(a, m, pre, post);
        else if (RB > 2 && p == 1) apply_u1_real<R, RB, 1 % RB, PRE, POST, ZIN>(a, m, pre, post);
        else if (RB > 3 && p == 2) apply_u1_real<R, RB, 2 % RB, PRE, POST, ZIN>(a, m, pre, post);
        else apply_u1_real<R, RB, RB - 1, PRE, POST, ZIN>(a, m, pre, post);
        return;
    }
    if (RB > 1 && p == 0) apply_u1<R, RB, 0, PRE, POST, ZIN>(a, m, pre, post);
    else if (RB > 2 && p == 1) apply_u1<R, RB, 1 % RB, PRE, POST, ZIN>(a, m, pre, post);
    else if (RB > 3 && p == 2) apply_u1<R, RB, 2 % RB, PRE, POST, ZIN>(a, m, pre, post);
    else apply_u1<R, RB, RB - 1, PRE, POST, ZIN>(a, m, pre, post);
}

// zin: 0 general, 1 the |1> inputs are zero (no input phase to apply), 2 the |0> inputs are zero.
// postkind: 0 no output block, 1 one factor per thread, 2 with register-bit factors.
template <typename R, int RB, int PRE, int ZIN>
__device__ __forceinline__ void dispatch_u1_post(int p, bool real, int postkind, tv<R> (&a)[1 << RB],
                                                 const cxf<R> (&m)[4], const PhaseSet<R, RB> &pre,
                                                 const PhaseSet<R, RB> &post)
{
    if (postkind == 2) dispatch_u1_pp<R, RB, PRE, 2, ZIN>(p, real, a, m, pre, post);
    else if (postkind == 1) dispatch_u1_pp<R, RB, PRE, 1, ZIN>(p, real, a, m, pre, post);
    else dispatch_u1_pp<R, RB, PRE, 0, ZIN>(p, real, a, m, pre, post);
}

template <typename R, int RB>
__device__ __forceinline__ void dispatch_u1(int p, bool real, int prekind, int zin, int postkind,
                                            tv<R> (&a)[1 << RB], const cxf<R> (&m)[4],
                                            const PhaseSet<R, RB> &pre, const PhaseSet<R, RB> &post)
{
    if (zin == 1) {
        dispatch_u1_post<R, RB, 0, 1>(p, real, postkind, a, m, pre, post);
    } else if (zin == 2) {
        if (prekind == 2) dispatch_u1_post<R, RB, 2, 2>(p, real, postkind, a, m, pre, post);
        else if (prekind == 1) dispatch_u1_post<R, RB, 1, 2>(p, real, postkind, a, m, pre, post);
        else dispatch_u1_post<R, RB, 0, 2>(p, real, postkind, a, m, pre, post);
    } else if (prekind == 2) {
        dispatch_u1_post<R, RB, 2, 0>(p, real, postkind, a, m, pre, post);
    } else if (prekind == 1) {
        dispatch_u1_post<R, RB, 1, 0>(p, real, postkind, a, m, pre, post);
    } else {
        dispatch_u1_post<R, RB, 0, 0>(p, real, postkind, a, m, pre, post);
    }
}

template <typename R, int RB, bool REAL>
__device__ __forceinline__ void dispatch_u2_t(int p0, int p1, tv<R> (&a)[1 << RB], const cxf<R> (&m)[16])
{
    if constexpr (RB >= 2) {
        switch (p0 * 4 + p1) {
#define QS_U2_CASE(A, B) \
    case (A) * 4 + (B): if constexpr ((A) < RB && (B) < RB) apply_u2<R, RB, (A) % RB, (B) % RB, REAL>(a, m); break;
        QS_U2_CASE(0, 1) QS_U2_CASE(1, 0) QS_U2_CASE(0, 2) QS_U2_CASE(2, 0)
        QS_U2_CASE(0, 3) QS_U2_CASE(3, 0) QS_U2_CASE(1, 2) QS_U2_CASE(2, 1)
        QS_U2_CASE(1, 3) QS_U2_CASE(3, 1) QS_U2_CASE(2, 3) QS_U2_CASE(3, 2)
#undef QS_U2_CASE
        default: break;
        }
    }
}

template <typename R, int RB>
__device__ __forceinline__ void dispatch_u2(int p0, int p1, bool real, tv<R> (&a)[1 << RB], const cxf<R> (&m)[16])
{
    if (real) dispatch_u2_t<R, RB, true>(p0, p1, a, m);
    else dispatch_u2_t<R, RB, false>(p0, p1, a, m);
}

}  // namespace qs
