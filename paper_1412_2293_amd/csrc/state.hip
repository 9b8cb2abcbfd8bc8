// Circuits on states that fit one CU's LDS: the whole circuit of a slot in one workgroup.
//
// Such a run is a serial chain of gates per slot.  Up to about 11 qubits its time is the latency of each
// step and not a rate: what a gate needs (its descriptor, matrix and phase tables) therefore comes from
// the LDS, staged once per stage for all its gates by coalesced loads, instead of from two dependent
// scalar loads per gate that miss the scalar cache (about 1 us per gate on one workgroup); the next
// gate's descriptor is read while this one runs.  At 13 and 14 qubits it is the vector issue of the one
// CU that holds the slot.  Registers hold 2^RB amplitudes per thread, few for small states, so that a
// slot's gates spread over the CU's four SIMDs; rounds exchange the state through the LDS, in two
// buffers taken in turn where that costs no workgroup (one barrier per exchange instead of two).
// Grover n = 10, complex<double>: 200 trajectories 512 us as passes, 154 us here; one 628 and 155.  Random
// pairs n = 14, 60 layers, 16 trajectories, complex<float>: 1.01 ms in 18 passes, 0.83 ms here.
#include <algorithm>
#include <cmath>

#include <type_traits>

#include "internal.h"
#include "regops.h"

namespace qs {

// Threads of a workgroup at most: complex<float> states of 14 qubits take 1024 of 16 amplitudes.
template <typename R, int RB>
constexpr int kStateThreads = (sizeof(R) == 4 && RB == 4) ? 1024 : 512;

__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ float uniform(float x) { return __uint_as_float(uniform(__float_as_uint(x))); }
__device__ __forceinline__ double uniform(double x)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const uint32_t lo = uniform((uint32_t)b), hi = uniform((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// PLAIN: every one-qubit op is real without phases and there is no two-qubit op (Grover).
template <typename R, int RB, bool PLAIN>
__global__ void __launch_bounds__((kStateThreads<R, RB>))
    k_state(R *__restrict__ psi, int n, int pass_index, int64_t init, const RunParams *__restrict__ dyn,
            const PassDesc *__restrict__ g_passes, const StageDesc *__restrict__ g_stages,
            const RoundDesc *__restrict__ g_rounds, const StateOp *__restrict__ g_sops,
            const cxf<R> *__restrict__ rec_all, int two_buffers)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NR = 1 << RB;
    const PassDesc *pd = g_passes + pass_index;
    // a tile of fewer threads than a wave runs in copies of them (which store the same values), so that a
    // whole wave stages the records (random pairs n = 2, 60 layers, 3001 slots, complex<float>: 940 us with
    // one thread per slot, 304 with 64)
    const uint32_t nthr = 1u << (n - RB), tid = threadIdx.x & (nthr - 1u), sid = threadIdx.x, stride = blockDim.x;
    const int slot = (int)blockIdx.x;
    if (dyn) init = dyn->init;
    const uint32_t tile_entries = 1u << n;
    cxf<R> *tile = reinterpret_cast<cxf<R> *>(smem);
    StateOp *lops = reinterpret_cast<StateOp *>(tile + ((size_t)tile_entries << two_buffers));
    cxf<R> *lrec = reinterpret_cast<cxf<R> *>(lops + kStageSops);
    const cxf<R> *rec = rec_all + (size_t)slot * pd->rec_size;

    // register layout: tile-local index of register r is lthr | the OR of the positions of r's bits
    uint32_t mask = g_rounds[pd->round_begin].reg_mask, pos[RB], lthr;
    auto set_layout = [&](uint32_t m) {
        mask = m;
        uint32_t x = tid;
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const uint32_t b = (uint32_t)__builtin_ctz(m);
            pos[k] = 1u << b;
            const uint32_t lo = x & (pos[k] - 1u);
            x = ((x ^ lo) << 1) | lo;
            m &= m - 1u;
        }
        lthr = x;
    };
    auto reg_off = [&](int r) {
        uint32_t o = 0;
#pragma unroll
        for (int k = 0; k < RB; ++k)
            if ((r >> k) & 1) o |= pos[k];
        return o;
    };
    set_layout(mask);
    tv<R> a[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) a[r] = tv<R>{(lthr | reg_off(r)) == (uint32_t)init ? (R)1 : (R)0, (R)0};
    uint32_t buf = 0;

    // the swizzle is linear over XOR: one per thread and one per register bit
    auto exchange = [&](uint32_t to) {
        uint32_t sw = lds_swizzle(lthr), sp[RB];
#pragma unroll
        for (int k = 0; k < RB; ++k) sp[k] = lds_swizzle(pos[k]);
        if (!two_buffers) __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            uint32_t o = 0;
#pragma unroll
            for (int k = 0; k < RB; ++k)
                if ((r >> k) & 1) o ^= sp[k];
            tile[buf + (sw ^ o)] = cx<R>(a[r]);
        }
        __syncthreads();
        set_layout(to);
        sw = lds_swizzle(lthr);
#pragma unroll
        for (int k = 0; k < RB; ++k) sp[k] = lds_swizzle(pos[k]);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            uint32_t o = 0;
#pragma unroll
            for (int k = 0; k < RB; ++k)
                if ((r >> k) & 1) o ^= sp[k];
            a[r] = tvec(tile[buf + (sw ^ o)]);
        }
        if (two_buffers) buf ^= tile_entries;
    };
    // Keeps the tile in one set of registers (no instructions): where branches update it, the compiler would give
    // each its own copy of a complex<double> tile, 165 registers for 8 amplitudes, and spills for 16 (random pairs
    // n = 12, 10 layers, 3001 slots: 1424 us with the copies, 1010 without).
    auto keep = [&]() {
        if constexpr (sizeof(R) == 8) {
#pragma unroll
            for (int r = 0; r < NR; ++r) asm volatile("" : "+v"(a[r]));
        }
    };
    // the factor of a folded block for this thread
    auto block_w = [&](uint32_t at, bool uni) {
        const cxf<R> *b = lrec + at;
        if (uni) return b[4];
        cxf<R> w = mul(b[4 + (tid & 31u)], b[36 + ((tid >> 5) & 15u)]);
        if (nthr > 512u) w = mul(w, b[52 + (tid >> 9)]);
        return w;
    };
    // |1> amplitudes of register bit P times the block's phases
    auto phases = [&](auto pc, uint32_t at, uint32_t kind, bool uni) {
        constexpr int P = decltype(pc)::value;
        PhaseSet<R, RB> ps;
        ps.w = block_w(at, uni);
        if (kind == 1u) {
#pragma unroll
            for (int k = 0; k < NR / 2; ++k) {
                const int r = pair_base<P>(k) | (1 << P);
                a[r] = tvec(mul(ps.w, cx<R>(a[r])));
            }
        } else {
#pragma unroll
            for (int k = 0; k < RB; ++k) ps.bit[k] = lrec[at + k];
#pragma unroll
            for (int k = 0; k < NR / 2; ++k) {
                const int r = pair_base<P>(k);
                a[r | (1 << P)] = tvec(mul(pair_phase<R, RB, P, true>(ps, r), cx<R>(a[r | (1 << P)])));
            }
        }
    };
    // the one-qubit op on register bit P; mr: its matrix's real parts, read ahead where they are kept
    constexpr bool kAhead = PLAIN || RB < 4;
    auto u1 = [&](auto pc, uint32_t w0, uint32_t w1, const R (&mr)[4]) {
        constexpr int P = decltype(pc)::value;
        const cxf<R> *rm = lrec + (w0 & 0xffffu);
        const uint32_t fl = w1 >> 16;
        if constexpr (!PLAIN)
            if (fl & 3u) phases(pc, w0 >> 16, fl & 3u, (fl & SOP_PRE_UNI) != 0);
        if (PLAIN || (fl & SOP_REAL)) {
            const R m0 = kAhead ? mr[0] : rm[0].re, m1 = kAhead ? mr[1] : rm[1].re, m2 = kAhead ? mr[2] : rm[2].re,
                    m3 = kAhead ? mr[3] : rm[3].re;
#pragma unroll
            for (int k = 0; k < NR / 2; ++k) {
                const int r = pair_base<P>(k);
                const tv<R> x0 = a[r], x1 = a[r | (1 << P)];
                a[r] = tv<R>{m0 * x0.x + m1 * x1.x, m0 * x0.y + m1 * x1.y};
                a[r | (1 << P)] = tv<R>{m2 * x0.x + m3 * x1.x, m2 * x0.y + m3 * x1.y};
            }
        } else {
            const cxf<R> m[4] = {rm[0], rm[1], rm[2], rm[3]};
            PhaseSet<R, RB> none;
            apply_u1<R, RB, P, 0, 0, 0>(a, m, none, none);
        }
        if constexpr (!PLAIN)
            if (fl & 12u) phases(pc, w1 & 0xffffu, (fl >> 2) & 3u, (fl & SOP_POST_UNI) != 0);
    };

    for (int si = pd->stage_begin; si < pd->stage_end; ++si) {
        const StageDesc *sd = g_stages + si;
        const int nops = sd->sop_end - sd->sop_begin;
        {
            // every wave is past the previous stage's records
            __syncthreads();
            const uint4 *src = reinterpret_cast<const uint4 *>(g_sops + sd->sop_begin);
            uint4 *dst = reinterpret_cast<uint4 *>(lops);
            const int chunks = nops * (int)(sizeof(StateOp) / 16);
            for (int i = (int)sid; i < chunks; i += (int)stride) dst[i] = src[i];
            const cxf<R> *rs = rec + sd->rec_begin;
            const int entries = sd->rec_end - sd->rec_begin;
            for (int i = (int)sid; i < entries; i += (int)stride) lrec[i] = rs[i];
            __syncthreads();
        }
        StateOp next = lops[0];
        for (int oi = 0; oi < nops; ++oi) {
            const uint32_t code = uniform(next.code), to = uniform(next.to), la = uniform(next.a), lb = uniform(next.b);
            uint32_t w[RB][2];
#pragma unroll
            for (int k = 0; k < RB; ++k) {
                w[k][0] = uniform(next.op[k][0]);
                w[k][1] = PLAIN ? 0u : uniform(next.op[k][1]);
            }
            next = lops[oi + 1 < nops ? oi + 1 : oi];
            // the matrices, so that their latency overlaps the exchange (absent ops read entry 0)
            R mr[RB][4];
#pragma unroll
            for (int k = 0; k < RB; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) mr[k][j] = kAhead ? lrec[(w[k][0] & 0xffffu) + j].re : (R)0;
            if (to) exchange(to);
            keep();
            const uint32_t kind = code & 3u;
            if (kind == SOP_SEQ) {
                if (code & 4u) u1(std::integral_constant<int, 0>{}, w[0][0], w[0][1], mr[0]);
                if constexpr (PLAIN) keep();
                if (code & 8u) u1(std::integral_constant<int, 1>{}, w[1][0], w[1][1], mr[1]);
                if constexpr (PLAIN) keep();
                if constexpr (RB > 2)
                    if (code & 16u) u1(std::integral_constant<int, 2>{}, w[2 % RB][0], w[2 % RB][1], mr[2 % RB]);
                if constexpr (PLAIN) keep();
                if constexpr (RB > 3)
                    if (code & 32u) u1(std::integral_constant<int, 3>{}, w[3 % RB][0], w[3 % RB][1], mr[3 % RB]);
            } else if (PLAIN || kind == SOP_DIAG) {
                // diagonal pattern on (tile-local index & la) == lb
                const bool hit = (lthr & la) == (lb & ~mask);
                const uint32_t rmask = la & mask, rval = lb & mask;
                const cxf<R> f = lrec[w[0][0] & 0xffffu];
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if ((reg_off(r) & rmask) == rval) {
                        const tv<R> y = tvec(mul(f, cx<R>(a[r])));
                        a[r] = hit ? y : a[r];
                    }
            } else if constexpr (!PLAIN) {
                cxf<R> m[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const cxf<R> x = lrec[(w[0][0] & 0xffffu) + k];
                    m[k].re = uniform(x.re);
                    m[k].im = uniform(x.im);
                }
                dispatch_u2<R, RB>((int)((code >> 2) & 3u), (int)((code >> 4) & 3u), ((w[0][1] >> 16) & SOP_REAL) != 0, a,
                                   m);
            }
        }
    }
    R *base = psi + ((uint64_t)slot << (n + 1));
#pragma unroll
    for (int r = 0; r < NR; ++r) *reinterpret_cast<tv<R> *>(base + 2 * (size_t)(lthr | reg_off(r))) = a[r];
}

size_t state_stage_bytes(qs_dtype dt, int n)
{
    return (size_t)kStageSops * sizeof(StateOp) + (size_t)stage_rec_cap(dt, n) * 2 * (dt == QS_C64 ? 4 : 8);
}

bool state_shape(qs_dtype dt, int n, int RB)
{
    if (RB < 2 || RB > kMaxRegBits || n < RB || n > kMaxTileBits) return false;
    const int threads_log = n - RB;
    if (threads_log > (dt == QS_C64 && RB == 4 ? 10 : 9)) return false;
    return fused_lds_bytes(dt, n) + state_stage_bytes(dt, n) <= 160 * 1024;
}

// Register bits of the automatic plan: the fewest whose workgroup is allowed and, up to 3, has at most 256
// threads (random layers, 50 trajectories: n = 12 complex<float> 334 us with 3 against 380 with 4, complex<double>
// 438 against 461; Grover n = 8 complex<double> 169 with 2, 197 with 3, 257 with 4.  Random pairs n = 11, 60
// layers, with 2 and with 3, complex<float>: 2 slots 425 us and 450, 3001 slots 2320 and 1860; complex<double>:
// 494 and 505, 3250 and 3050).
int state_reg_bits(qs_dtype dt, int n)
{
    for (int rb = 2; rb <= kMaxRegBits; ++rb)
        if (state_shape(dt, n, rb) && (rb >= 3 || n - rb <= 8)) return rb;
    return 0;
}

// One-time opt-in to the full 160 KiB of LDS, which also notes the waves per CU that the variant's registers
// allow.
template <typename R, int RB, bool PLAIN>
static int state_waves = 0;

template <typename R, int RB, bool PLAIN>
static hipError_t state_attr_one()
{
    static const hipError_t attr = [] {
        hipFuncAttributes fa;
        const hipError_t e = hipFuncGetAttributes(&fa, (const void *)k_state<R, RB, PLAIN>);
        if (e != hipSuccess) return e;
        state_waves<R, RB, PLAIN> = 4 * std::min(8, 512 / std::max(fa.numRegs, 1));
        return hipFuncSetAttribute((const void *)k_state<R, RB, PLAIN>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   160 * 1024);
    }();
    return attr;
}

// Whether the state is exchanged through two LDS buffers in turn (one barrier per exchange) or one (two
// barriers).  Two where every slot's workgroup runs at once with two buffers, or where the registers admit no
// more workgroups to a CU with one; else one, so that more workgroups share a CU (random pairs n = 13, 10
// layers, 3001 slots, complex<float>: 1298 us with two, 985 with one; n = 8 297 and 253; n = 11,
// complex<double>, where the registers admit two either way, Grover: 638 and 671).  The results are the same.
static bool state_two_buffers(size_t tile, size_t stage, int threads, int waves, int S)
{
    constexpr size_t lds = 160 * 1024;
    constexpr int cus = 256;
    if (2 * tile + stage > lds) return false;
    const int by_regs = waves * 64 / threads;
    const int two = std::min((int)(lds / (2 * tile + stage)), by_regs), one = std::min((int)(lds / (tile + stage)), by_regs);
    return one <= two || S <= cus * two;
}

template <typename R, int RB, bool PLAIN>
static hipError_t state_launch_t(R *psi, qs_dtype dt, int n, int S, int pass_index, int64_t init, const RunParams *dyn,
                                 ProgramDev prog, const void *rec, hipStream_t st)
{
    const hipError_t attr = state_attr_one<R, RB, PLAIN>();
    if (attr != hipSuccess) return attr;
    const size_t tile = fused_lds_bytes(dt, n), stage = state_stage_bytes(dt, n);
    const unsigned threads = std::max(64u, 1u << (n - RB));
    const int two = state_two_buffers(tile, stage, (int)threads, state_waves<R, RB, PLAIN>, S) ? 1 : 0;
    hipLaunchKernelGGL((k_state<R, RB, PLAIN>), dim3((unsigned)S), dim3(threads), (tile << two) + stage, st, psi, n, pass_index,
                       init, dyn, prog.passes, prog.stages, prog.rounds, prog.sops, (const cxf<R> *)rec, two);
    return hipGetLastError();
}

hipError_t state_prepare_attributes()
{
    hipError_t e = hipSuccess;
#define QS_STATE_ATTR(R, RB)                                          \
    if (e == hipSuccess) e = state_attr_one<R, RB, false>();          \
    if (e == hipSuccess) e = state_attr_one<R, RB, true>();
    QS_STATE_ATTR(float, 2) QS_STATE_ATTR(float, 3) QS_STATE_ATTR(float, 4)
    QS_STATE_ATTR(double, 2) QS_STATE_ATTR(double, 3) QS_STATE_ATTR(double, 4)
#undef QS_STATE_ATTR
    return e;
}

hipError_t launch_state_pass(void *psi, qs_dtype dt, int n, int S, const PassDesc *h, int pass_index, int64_t init,
                             ProgramDev prog, const void *rec, hipStream_t st, const RunParams *dyn)
{
    if (!h->state || h->K != n || init < 0 || !state_shape(dt, n, h->RB)) return hipErrorInvalidValue;
    TimedLaunch tl("fused", (double)S * std::ldexp(1.0, n) * amp_bytes(dt), st);
#define QS_STATE_RUN(R, RB, PLAIN)                                                                                   \
    state_launch_t<R, RB, PLAIN>((R *)psi, dt, n, S, pass_index, init, dyn, prog, rec, st)
#define QS_STATE_CASE(RB)                                                                                            \
    case RB:                                                                                                        \
        if (h->state == 2)                                                                                          \
            return dt == QS_C64 ? QS_STATE_RUN(float, RB, true) : QS_STATE_RUN(double, RB, true);                   \
        return dt == QS_C64 ? QS_STATE_RUN(float, RB, false) : QS_STATE_RUN(double, RB, false);
    switch (h->RB) {
        QS_STATE_CASE(2)
        QS_STATE_CASE(3)
        QS_STATE_CASE(4)
    }
#undef QS_STATE_CASE
#undef QS_STATE_RUN
    return hipErrorInvalidValue;
}

}  // namespace qs
