// Expanding passes of the fused program.
#include "cplx.h"
#include "internal.h"

#include <cmath>

namespace qs {

// ---------------------------------------------------------------------------------------
// Expanding passes (PassDesc::expand): every op is a real 2 x 2 update of a target that still
// holds its basis bit, with at most one uniform output phase w.  One input of each pair is zero,
// so the op multiplies the other by A (output bit 0) or B w (output bit 1), and the whole pass is
//   out(l) = in(l with the targets at their basis bits) * prod over targets t of c_t[bit t of l],
// c_t = (A_t, B_t w_t): one product per amplitude instead of one update per op and an exchange
// through the LDS per four ops.  What is left is the store of the state (write bound).
//
// The product is split over the index bits a thread's amplitudes share: tables of the factors of
// thread bits 0..3 (with the vector's bit 0 in complex<float>) and 4..7, formed once per
// workgroup and slot in FP64 and rounded once, a per-thread base (their product times the
// input), and the products of the register bits.  A workgroup takes up to kExpandSlots slots of a
// tile: the latency of its set-up is paid once for them, and slot 0's amplitudes, which the
// overlaps need, are formed once for them (reading them back cost 0.07 ms per 128 MiB of them).
// All inputs of a tile are read before the barrier that precedes its first store, the next tile's
// while this one is stored.
// QFT n = 26, complex<float>, 17 slots (9.1 GB written): the last pass 3.48 + 0.25 ms as updates,
// 1.65 + 0.11 ms here, 5.2 TB/s of stores (a fill of one buffer reaches 6.9; without its stores
// the pass takes 0.52 ms).  One slot per workgroup: 2.8 ms; two: 2.0.
// ---------------------------------------------------------------------------------------
// Factors of an expanding pass: record entries 2j and 2j + 1 of a slot are the factors of
// tile-local bit j for the output bits 0 and 1 ((1, 1) for a bit that is no target).  One wave per
// (slot, tile-local bit): the lanes take the folded phases, at most one per qubit, and multiply
// them in a tree.  Phases conditioned on tile-number bits go to their record entries.
template <typename R>
__global__ void __launch_bounds__(256)
    k_expand_prep(int S, int pass_index, const PassDesc *__restrict__ passes, const OpDesc *__restrict__ ops,
                  const PrepRef *__restrict__ prefs, const double *__restrict__ tab, cxf<R> *__restrict__ rec_all,
                  uint64_t basis, const RunParams *__restrict__ dyn)
{
    const PassDesc *pd = passes + pass_index;
    const int K = pd->K, lane = (int)(threadIdx.x & 63u);
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= (int64_t)S * K) return;
    if (dyn) basis = (uint64_t)dyn->init;
    const int slot = (int)(w / K), j = (int)(w % K);
    cxf<R> *rec = rec_all + (size_t)slot * pd->rec_size;
    const int o = pd->xop[j];
    if (o < 0) {
        if (lane < 2) rec[2 * j + lane] = cxf<R>{(R)1, (R)0};
        return;
    }
    const OpDesc *op = ops + pd->op_begin + o;
    double2 ph = make_double2(1.0, 0.0);
    for (int k = op->pref_begin + lane; k < op->pref_end; k += 64) {
        const PrepRef pr = prefs[k];
        const double *t = tab + ((uint64_t)pr.gate * S + slot) * 8;
        const double2 v = make_double2(t[0], t[1]);
        if (pr.kind == PR_OUTER) rec[pr.slot_entry] = cxf<R>{(R)v.x, (R)v.y};
        else if ((basis >> pr.bit) & 1ull) ph = dmul(ph, v);   // PR_BASIS, the only other kind here
    }
    for (int off = 32; off > 0; off >>= 1)
        ph = dmul(ph, make_double2(__shfl_xor(ph.x, off, 64), __shfl_xor(ph.y, off, 64)));
    if (lane < 2) {
        const int b1 = (int)((basis >> pd->q_pos[j]) & 1ull);
        const double m = tab[((uint64_t)op->gate * S + slot) * 8 + 4 * lane + 2 * b1];
        rec[2 * j + lane] = lane ? cxf<R>{(R)(m * ph.x), (R)(m * ph.y)} : cxf<R>{(R)m, (R)0};
    }
}

hipError_t launch_expand_prep(qs_dtype dt, int S, const PassDesc *h, int pass_index, ProgramDev prog, const double *tab,
                              void *rec, int64_t basis, const RunParams *dyn, hipStream_t st)
{
    TimedLaunch tl("prep", (double)S * 2 * h->K * (dt == QS_C64 ? 8 : 16), st);
    const unsigned blocks = (unsigned)(((int64_t)S * h->K + 3) / 4);
    if (dt == QS_C64)
        hipLaunchKernelGGL(k_expand_prep<float>, dim3(blocks), dim3(256), 0, st, S, pass_index, prog.passes, prog.ops,
                           prog.prefs, tab, (cxf<float> *)rec, (uint64_t)basis, dyn);
    else
        hipLaunchKernelGGL(k_expand_prep<double>, dim3(blocks), dim3(256), 0, st, S, pass_index, prog.passes, prog.ops,
                           prog.prefs, tab, (cxf<double> *)rec, (uint64_t)basis, dyn);
    return hipGetLastError();
}

// OVL: 0 no overlaps, 1 slot 0 itself (its squared norm), 2 the other slots, before slot 0: its
// amplitudes are formed from its inputs beside theirs, with the same operations that later store
// them, instead of being read back.
template <typename R, int OVL>
__global__ void __launch_bounds__(256, 4)
    k_expand(R *__restrict__ psi, int n, int pass_index, int64_t init, int64_t basis, const RunParams *__restrict__ dyn,
             const PassDesc *__restrict__ g_passes, const OpDesc *__restrict__ g_ops, const cxf<R> *__restrict__ rec_all,
             const cxf<R> *__restrict__ wtab, const uint64_t *__restrict__ otab, double *__restrict__ ovl, int slot_base,
             int slots, int per, int groups, int run)
{
    constexpr int VB = sizeof(R) == 4 ? 1 : 0, V = 1 << VB;   // amplitudes per 16-byte vector
    constexpr int RBX = kExpandRegs - VB, NRX = 1 << RBX;
    constexpr int G = kExpandSlots, GT = G + (OVL == 2 ? 1 : 0);   // GT - 1: slot 0
    __shared__ cxf<R> F[GT][24], T1[GT][V][16], T2[GT][16], TP[GT][NRX];
    __shared__ double red[OVL ? G : 1][3][4];   // the waves' sums
    const PassDesc *pd = g_passes + pass_index;
    const int K = pd->K;
    if (dyn) {
        basis = dyn->init;
        if (init >= 0) init = basis;
    }
    const int tiles_log = __builtin_popcountll(pd->outer_mask & ~pd->classical);
    uint64_t tile = blockIdx.x / (unsigned)groups * (uint64_t)run;   // the first of `run` tiles
    const int s0 = slot_base + (int)(blockIdx.x % (unsigned)groups) * per;
    const int left = slot_base + slots - s0, cnt = left < per ? left : per;
    const uint32_t tid = threadIdx.x, nthr = blockDim.x;
    const int n_jobs = pd->job_end - pd->job_begin;
    // targets, register bits (the highest targets) and thread bits of the tile-local index
    uint32_t tmask = 0, blocal = 0, rmask = 0;
    for (int j = 0; j < K; ++j) {
        if (pd->xop[j] >= 0) tmask |= 1u << j;
        if (((uint64_t)basis >> pd->q_pos[j]) & 1ull) blocal |= 1u << j;
    }
    int rpos[RBX];
    {
        uint32_t m = tmask;
#pragma unroll
        for (int k = RBX - 1; k >= 0; --k) {
            rpos[k] = 31 - __builtin_clz(m);
            m ^= 1u << rpos[k];
            rmask |= 1u << rpos[k];
        }
    }
    const uint32_t thr_mask = ((1u << K) - 1u) & ~rmask & ~(uint32_t)VB;

    // the factors of every tile-local bit, with this tile's products of the phases conditioned on
    // tile-number bits: all loads at once, then the products from the LDS
    auto slot_of = [&](int s) { return s == G ? 0 : s0 + (s < cnt ? s : cnt - 1); };   // repeats beyond the last
    for (int x = (int)tid; x < GT * 2 * K; x += (int)nthr) {
        const int s = x / (2 * K), e = x % (2 * K), slot = slot_of(s);
        cxf<R> f = rec_all[(size_t)slot * pd->rec_size + e];
        const int o = pd->xop[e >> 1];
        if (n_jobs > 0 && (e & 1) && o >= 0) {
            const int job = g_ops[pd->op_begin + o].post_job;
            if (job >= 0) f = mul(f, wtab[(((uint64_t)slot << tiles_log) | tile) * (size_t)n_jobs + job]);
        }
        F[s][e] = f;
    }
    __syncthreads();
    constexpr int E = 16 * V + 16 + NRX;
    for (int x = (int)tid; x < GT * E; x += (int)nthr) {
        const int s = x / E, e = x % E;
        auto factor = [&](int j, uint32_t bit) {
            const cxf<R> f = F[s][2 * j + (int)bit];
            return make_double2((double)f.re, (double)f.im);
        };
        double2 f = make_double2(1.0, 0.0);
        if (e < 16 * V + 16) {
            const int hi = e >= 16 * V;   // thread bits 4..7
            const uint32_t y = hi ? (uint32_t)(e - 16 * V) : (uint32_t)e & 15u;
            uint32_t m = thr_mask;
            for (int k = 0; k < 4 * hi; ++k) m &= m - 1u;
            for (int k = 0; k < 4 && m; ++k) {
                f = dmul(f, factor(__builtin_ctz(m), (y >> k) & 1u));
                m &= m - 1u;
            }
            if (VB && !hi) f = dmul(f, factor(0, (uint32_t)e >> 4));
            const cxf<R> v = {(R)f.x, (R)f.y};
            if (hi) T2[s][y] = v;
            else T1[s][e >> 4][y] = v;
        } else {
            const int y = e - 16 * V - 16;
            uint32_t m = rmask;
            for (int k = 0; k < RBX; ++k) {
                f = dmul(f, factor(__builtin_ctz(m), (uint32_t)(y >> k) & 1u));
                m &= m - 1u;
            }
            TP[s][y] = cxf<R>{(R)f.x, (R)f.y};
        }
    }
    // this thread's amplitudes: tile-local index lthr | v | register bits
    const uint32_t lthr = deposit32(tid, thr_mask, K);
    uint64_t pst = 0, pin = 0;
    for (int j = 0; j < K; ++j) {
        const uint64_t b = 1ull << pd->q_pos[j];
        if ((lthr >> j) & 1u) pst |= b;
        if (((((tmask >> j) & 1u) ? blocal : lthr) >> j) & 1u) pin |= b;
    }
    // inputs: zero unless the non-target bits agree with the basis where no gate has touched them
    const uint32_t lc = pd->lclassical & ~tmask;
    const bool vt = VB && (tmask & 1u);                // bit 0 a target: one input for both
    bool ok[V];
#pragma unroll
    for (int v = 0; v < V; ++v) ok[v] = (((vt ? lthr : lthr | (uint32_t)v) ^ blocal) & lc) == 0;
    uint64_t rbit[RBX];
#pragma unroll
    for (int k = 0; k < RBX; ++k) rbit[k] = 1ull << pd->q_pos[rpos[k]];
    typedef R vec __attribute__((ext_vector_type(2 * V)));
    auto slot_ptr = [&](int s) { return psi + ((uint64_t)slot_of(s) << (n + 1)); };
    cxf<R> in[GT][V];
    auto load_in = [&](uint64_t outer) {
        const uint64_t gin = outer | pin;
#pragma unroll
        for (int s = 0; s < GT; ++s)
#pragma unroll
            for (int v = 0; v < V; ++v) in[s][v] = cxf<R>{(R)0, (R)0};
        if (init >= 0) {
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (ok[v] && (vt ? gin : gin | (uint64_t)v) == (uint64_t)init)
#pragma unroll
                    for (int s = 0; s < GT; ++s) in[s][v].re = (R)1;
        } else if (ok[0] || ok[V - 1]) {
#pragma unroll
            for (int s = 0; s < GT; ++s)
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    // (the vector's other amplitude where the input is not to be read)
                    const uint64_t gi = vt ? gin : gin | (uint64_t)(ok[v] ? v : V - 1 - v);
                    const cxf<R> x = *reinterpret_cast<const cxf<R> *>(slot_ptr(s) + 2 * gi);
                    in[s][v] = ok[v] ? x : cxf<R>{(R)0, (R)0};
                }
        }
    };
    double sum[OVL ? G : 1][3];
#pragma unroll
    for (int s = 0; s < (OVL ? G : 1); ++s)
#pragma unroll
        for (int k = 0; k < 3; ++k) sum[s][k] = 0.0;
    uint64_t outer = otab[tile];
    load_in(outer);
    __syncthreads();
    for (int tt = 0; tt < run; ++tt) {
        cxf<R> b[GT][V];
#pragma unroll
        for (int s = 0; s < GT; ++s) {
            const cxf<R> t2 = T2[s][(tid >> 4) & 15u];
#pragma unroll
            for (int v = 0; v < V; ++v) b[s][v] = mul(mul(T1[s][v][tid & 15u], t2), in[s][v]);
        }
        const uint64_t gst = outer | pst;
        // every input of this tile has been read (its stores follow); the next tile's are loaded
        // while it is stored
        __syncthreads();
        if (tt + 1 < run) {
            outer = otab[tile + tt + 1];
            load_in(outer);
        }
#pragma unroll
        for (int r = 0; r < NRX; ++r) {
            uint64_t g = gst;
#pragma unroll
            for (int k = 0; k < RBX; ++k)
                if ((r >> k) & 1) g |= rbit[k];
            double ar[V], ai[V];
            if constexpr (OVL == 2) {
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const cxf<R> y = mul(b[GT - 1][v], TP[GT - 1][r]);
                    ar[v] = y.re;
                    ai[v] = y.im;
                }
            }
#pragma unroll
            for (int s = 0; s < G; ++s) {
                if (s >= cnt) break;
                const cxf<R> p = TP[s][r];
                vec o;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const cxf<R> y = mul(b[s][v], p);
                    o[2 * v] = y.re;
                    o[2 * v + 1] = y.im;
                    if constexpr (OVL > 0) {
                        const double br = y.re, bi = y.im;
                        sum[s][2] = __builtin_fma(bi, bi, __builtin_fma(br, br, sum[s][2]));
                        if constexpr (OVL == 2) {
                            sum[s][0] = __builtin_fma(ai[v], bi, __builtin_fma(ar[v], br, sum[s][0]));
                            sum[s][1] = __builtin_fma(-ai[v], br, __builtin_fma(ar[v], bi, sum[s][1]));
                        }
                    }
                }
                __builtin_nontemporal_store(o, reinterpret_cast<vec *>(slot_ptr(s) + 2 * g));
            }
        }
    }
    if constexpr (OVL > 0) {
        // sums over the lanes, then over the waves (fixed order, whatever the slots of the block)
#pragma unroll
        for (int s = 0; s < G; ++s) {
            if (s >= cnt) break;
            if constexpr (OVL == 1) sum[s][0] = sum[s][2];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                double t = sum[s][k];
                for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
                if ((tid & 63u) == 0) red[s][k][tid >> 6] = t;
            }
        }
        __syncthreads();
        if (tid < (uint32_t)cnt * 3u) {
            const int s = (int)tid / 3, k = (int)tid % 3;
            double t = 0.0;
            for (uint32_t w = 0; w < (nthr >> 6); ++w) t += red[s][k][w];
            ovl[((((uint64_t)(s0 + s) << tiles_log) | tile) / (uint64_t)run) * 3 + (uint64_t)k] = t;
        }
    }
}

// Log2 of the tiles per workgroup: two share the factor tables and the sums of the overlaps where
// that leaves a launch of one slot eight workgroups per CU, unless the tables depend on the tile
// (QFT n = 26, slot 0's launch: 109 us with two, 125 with one, 106 with four; 16 slots: 1.65, 1.64
// and 1.75 ms).  A function of the pass alone: a slot's partial sums do not depend on the other
// slots of the launch.
static int expand_run_log(int n, const PassDesc *h, int64_t init)
{
    if (h->job_end > h->job_begin) return 0;
    return fused_walked_bits(n, h, init) >= 12 ? 1 : 0;
}

int fused_partial_bits(int n, const PassDesc *h, int64_t init)
{
    return fused_walked_bits(n, h, init) - (h->expand ? expand_run_log(n, h, init) : 0);
}

hipError_t launch_expand_pass(void *psi, qs_dtype dt, int n, int S, const PassDesc *pass_host, int pass_index,
                              int64_t init, int64_t basis, ProgramDev prog, const void *rec, const void *wtab,
                              const uint64_t *otab, hipStream_t st, const RunParams *dyn, double *ovl, int slot_base,
                              int slots)
{
    const PassDesc &h = *pass_host;
    if (!h.expand || h.K < 10 || h.K > 12 || (init >= 0 && h.zero_fill) || basis < 0) return hipErrorInvalidValue;
    if (ovl && (slots < 1 || slot_base < 0 || slot_base + slots > S)) return hipErrorInvalidValue;
    if (!ovl) {
        slot_base = 0;
        slots = S;
    }
    const uint64_t tiles = 1ull << fused_walked_bits(n, pass_host, init);
    const int run = 1 << expand_run_log(n, pass_host, init);
    // as many slots per workgroup as leave four workgroups per CU
    int per = kExpandSlots;
    while (per > 1 && (tiles / run) * (uint64_t)((slots + per - 1) / per) < 1024) per >>= 1;
    const unsigned groups = (unsigned)((slots + per - 1) / per);
    const double tiles_share = std::ldexp(1.0, -__builtin_popcountll(h.classical));
    const double read_share = init >= 0 ? 0.0 : std::ldexp(1.0, -__builtin_popcount(h.lclassical));
    const double ref_share = ovl && slot_base > 0 ? 1.0 : 0.0;
    TimedLaunch tl("fused",
                   ((1.0 + read_share) * (double)slots + ref_share) * tiles_share * std::ldexp(1.0, n) * amp_bytes(dt),
                   st);
#define QS_EXPAND(R, OVL)                                                                                            \
    hipLaunchKernelGGL((k_expand<R, OVL>), dim3((unsigned)(tiles / run * groups)), dim3(1u << (h.K - 4)), 0, st, (R *)psi, \
                       n, pass_index, init, basis, dyn, prog.passes, prog.ops, (const cxf<R> *)rec,                  \
                       (const cxf<R> *)wtab, otab, ovl, slot_base, slots, per, (int)groups, run)
    if (dt == QS_C64) {
        if (!ovl) QS_EXPAND(float, 0);
        else if (slot_base == 0) QS_EXPAND(float, 1);
        else QS_EXPAND(float, 2);
    } else {
        if (!ovl) QS_EXPAND(double, 0);
        else if (slot_base == 0) QS_EXPAND(double, 1);
        else QS_EXPAND(double, 2);
    }
#undef QS_EXPAND
    return hipGetLastError();
}

}  // namespace qs
