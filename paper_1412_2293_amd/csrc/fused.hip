// Fused passes: the per-slot records, phase chains and per-tile tables that a pass reads, and its
// launch (the pass kernel itself is in fused_kernel.h).
#include <cmath>

#include "cplx.h"
#include "internal.h"

namespace qs {

template <typename R>
hipError_t fused_attributes();
template <typename R>
hipError_t fused_launch(R *p, int n, int S, const PassDesc &h, int pass_index, int rec_cap, int64_t init, int64_t basis,
                        const RunParams *dyn, ProgramDev prog, const void *rec, const void *wtab, const uint64_t *otab,
                        size_t lds, hipStream_t st, double *ovl, int slot_base, int slots);

// ---------------------------------------------------------------------------------------
// Per-slot records of one pass (one thread per op and slot; FP64 products rounded once).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double2 dconj(double2 a) { return make_double2(a.x, -a.y); }

// a / |a| (1 for a == 0)
__device__ __forceinline__ double2 dunit(double2 a)
{
    const double h = hypot(a.x, a.y);
    return h > 0.0 ? make_double2(a.x / h, a.y / h) : make_double2(1.0, 0.0);
}

// Per (slot, block round, column): column `col` of the round's block U (the ops applied in order
// to the basis state col, in FP64: each op's phases conditioned on register bits on its |1> input,
// its 2 x 2 matrix, the same on its output), written into the operand table with rows permuted
// as block_apply expects.  The matrices and register-bit factors come from the slot's records,
// written by k_pass_prep before.
template <typename R>
__global__ void k_block_prep(int S, int round_begin, int n_rounds, int rec_size, ProgramDev prog,
                             cxf<R> *__restrict__ rec_all)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)S * n_rounds * 16) return;
    const int col = (int)(t & 15);
    const int rr = (int)((t >> 4) % n_rounds);
    const int slot = (int)((t >> 4) / n_rounds);
    const RoundDesc &rd = prog.rounds[round_begin + rr];
    if (rd.block_rec < 0) return;
    cxf<R> *rec = rec_all + (size_t)slot * rec_size;
    double2 v[16];
    for (int b = 0; b < 16; ++b) v[b] = make_double2(b == col ? 1.0 : 0.0, 0.0);
    auto ld = [&](int e) { return make_double2((double)rec[e].re, (double)rec[e].im); };
    auto bit_phases = [&](int block, int p) {
        if (block < 0) return;
        double2 f[4];
        for (int k = 0; k < 4; ++k) f[k] = ld(block + k);
        for (int b = 0; b < 16; ++b) {
            if (!((b >> p) & 1)) continue;
            double2 w = make_double2(1.0, 0.0);
            for (int k = 0; k < 4; ++k)
                if (k != p && ((b >> k) & 1)) w = dmul(w, f[k]);
            v[b] = dmul(w, v[b]);
        }
    };
    for (int oi = rd.op_begin; oi < rd.op_end; ++oi) {
        const OpDesc &op = prog.ops[oi];
        const int p = op.p0;
        bit_phases(op.pre_rec, p);
        const double2 m0 = ld(op.rec), m1 = ld(op.rec + 1), m2 = ld(op.rec + 2), m3 = ld(op.rec + 3);
        for (int b = 0; b < 16; ++b) {
            if ((b >> p) & 1) continue;
            const double2 x0 = v[b], x1 = v[b | (1 << p)];
            const double2 y0 = dmul(m0, x0), y0b = dmul(m1, x1), y1 = dmul(m2, x0), y1b = dmul(m3, x1);
            v[b] = make_double2(y0.x + y0b.x, y0.y + y0b.y);
            v[b | (1 << p)] = make_double2(y1.x + y1b.x, y1.y + y1b.y);
        }
        bit_phases(op.post_rec, p);
    }
    // U[g][col] = v[g] goes to row P(g) of the permuted block; real form entries
    // (r, c) -> lane (r % 16) + 16 (c % 4), entry (r / 16) * 8 + c / 4 of the lane's 16
    R *tab = reinterpret_cast<R *>(rec + rd.block_rec);
    auto put = [&](int r, int c, double x) { tab[((r & 15) + 16 * (c & 3)) * 16 + (r >> 4) * 8 + (c >> 2)] = (R)x; };
    for (int g = 0; g < 16; ++g) {
        const int r = ((g & 3) << 2) | (g >> 2);
        put(r, col, v[g].x);
        put(r, 16 + col, -v[g].y);
        put(16 + r, col, v[g].y);
        put(16 + r, 16 + col, v[g].x);
    }
}

// ---------------------------------------------------------------------------------------
// Phase chains (W lanes per chain and slot, FP64).  Along a chain of one-qubit gates on
// one wire, each inner gate's matrix M (with the phase c carried from the gate before it
// multiplied into its |1> column) is factored as M = p * diag(1, b) * Rm * diag(1, d) with
// unit p, b, d and Rm real.  Its row is rewritten as Rm in words 0, 2, 4, 6 and the input
// phase d in words 1, 3; b is carried to the next gate, p into the global phase, which the
// last gate of the chain takes along with the carried b (its row stays a complex matrix).
// The factors: p = phase(M00), d = c phase(M01) / p, and b from the larger of the second row's
// entries, phase(M11) / phase(M01) or -phase(M10) / p; Rm is the real part of M with those phases
// divided out.  For a unitary M (M10 = -e^{it} conj(M01), M11 = e^{it} conj(M00)) the
// divided-out entries are real, so the factors reproduce M; a phase taken from a zero or
// rounding-sized entry only affects entries of that size.  (phase(0) = 1.)
// c drops out of b, so the lanes factor W gates at once, take c from the lane before and multiply
// the global phase in a tree (60 gates, 64 lanes: 74 us as one thread's walk, 4 us here).  The fewest
// lanes that hold the longest chain are taken: 42014 chains of 10 gates, 38 us with 64 lanes each and 17
// with 16.  A wider tree would only multiply by ones, so the results do not depend on W.
// ---------------------------------------------------------------------------------------
template <int W>
__global__ void __launch_bounds__(256) k_phase_chains(double *tab, int S, const int32_t *__restrict__ chain_gates,
                                                      const int32_t *__restrict__ chain_off, int n_chains)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / W;
    if (i >= (int64_t)n_chains * S) return;
    const int lane = (int)threadIdx.x % W;
    const int c = (int)(i / S), s = (int)(i % S);
    const int kb = chain_off[c], ke = chain_off[c + 1];
    const double2 one = make_double2(1.0, 0.0);
    double2 carry = one, glob = one;
    for (int k0 = kb; k0 < ke; k0 += W) {
        const int k = k0 + lane;
        const bool in = k < ke, inner = k < ke - 1;
        double *t = tab + ((int64_t)chain_gates[in ? k : ke - 1] * S + s) * 8;
        const double2 m00 = make_double2(t[0], t[1]), m01 = make_double2(t[2], t[3]);
        const double2 m10 = make_double2(t[4], t[5]), m11 = make_double2(t[6], t[7]);
        const double2 p = dunit(m00), q = dunit(m01);
        const double2 b = hypot(m11.x, m11.y) >= hypot(m10.x, m10.y)
                              ? dmul(dunit(m11), dconj(q))
                              : dmul(make_double2(-1.0, 0.0), dmul(dunit(m10), dconj(p)));
        double2 cin = make_double2(__shfl_up(b.x, 1, W), __shfl_up(b.y, 1, W));
        if (lane == 0) cin = carry;
        double2 g = inner ? p : one;
        for (int off = W / 2; off > 0; off >>= 1)
            g = dmul(g, make_double2(__shfl_xor(g.x, off, W), __shfl_xor(g.y, off, W)));
        glob = dmul(glob, g);
        if (inner) {
            const double2 d = dmul(cin, dmul(q, dconj(p))), pb = dmul(p, b);
            t[0] = dmul(m00, dconj(p)).x;
            t[2] = dmul(m01, dconj(q)).x;
            t[4] = dmul(m10, dconj(pb)).x;
            t[6] = dmul(m11, dconj(dmul(q, b))).x;
            t[1] = d.x;
            t[3] = d.y;
            t[5] = 0.0;
            t[7] = 0.0;
        } else if (in) {
            // the last gate: its chunk is the last one, so glob is complete
            const double2 gc = dmul(glob, cin);
            const double2 o[4] = {dmul(glob, m00), dmul(gc, m01), dmul(glob, m10), dmul(gc, m11)};
            for (int j = 0; j < 4; ++j) {
                t[2 * j] = o[j].x;
                t[2 * j + 1] = o[j].y;
            }
        }
        carry = make_double2(__shfl(b.x, W - 1, W), __shfl(b.y, W - 1, W));
    }
}

hipError_t launch_phase_chains(double *tab, int S, const int32_t *chain_gates, const int32_t *chain_off,
                               int n_chains, int longest, hipStream_t st)
{
    const int64_t tot = (int64_t)n_chains * S;
    if (tot <= 0) return hipSuccess;
    TimedLaunch tl("chains", (double)tot * 64.0, st);
#define QS_CHAINS(W)                                                                                          \
    hipLaunchKernelGGL(k_phase_chains<W>, dim3((unsigned)((tot * W + 255) / 256)), dim3(256), 0, st, tab, S,  \
                       chain_gates, chain_off, n_chains)
    if (longest <= 8) QS_CHAINS(8);
    else if (longest <= 16) QS_CHAINS(16);
    else if (longest <= 32) QS_CHAINS(32);
    else QS_CHAINS(64);
#undef QS_CHAINS
    return hipGetLastError();
}

// Per (slot, tile, outer job) of one pass: the product of the job's record entries whose
// tile-number bit is set in the tile's index, in the order the planner listed them.  Tiles are
// numbered as the fused kernel's blocks are (the walked tile-number bits, the others at their
// basis values), so a block finds its products at wtab + blockIdx * jobs.
// Also writes otab[tile]: the tile's tile-number bits of the physical index (the walked bits
// from the tile number, the others at the basis values), from the threads of slot 0, job 0.
// blockIdx.y: the pass, pass0 + blockIdx.y of the program, with its own areas (PassAreas).
template <typename R>
__global__ void k_pass_jobs(int S, int pass0, int fill_first, uint64_t basis, const PassDesc *__restrict__ passes,
                            const OuterJob *__restrict__ all_jobs, const int32_t *__restrict__ obits,
                            const char *__restrict__ rec_base, const RunParams *dyn, char *__restrict__ wt_base,
                            PassAreas ar)
{
    const PassDesc *pd = passes + pass0 + blockIdx.y;
    const int n_jobs = pd->job_end - pd->job_begin, rec_size = pd->rec_size;
    const bool fill = pass0 + (int)blockIdx.y == 0 && fill_first && pd->zero_fill;
    const uint64_t walk = fill ? pd->outer_mask : (pd->outer_mask & ~pd->classical);
    const int tiles_log = __builtin_popcountll(walk);
    const uint64_t classical = fill ? 0 : pd->classical;
    uint64_t fixed_bits = basis & classical;
    const OuterJob *__restrict__ jobs = all_jobs + pd->job_begin;
    const cxf<R> *__restrict__ rec_all = reinterpret_cast<const cxf<R> *>(rec_base + blockIdx.y * ar.rec_stride);
    uint64_t *__restrict__ otab = reinterpret_cast<uint64_t *>(wt_base + blockIdx.y * ar.wt_stride);
    cxf<R> *__restrict__ wtab = reinterpret_cast<cxf<R> *>(wt_base + blockIdx.y * ar.wt_stride + ar.otab_bytes);
    // thread order (slot, job, tile): the threads of a wave share the job, so its descriptor,
    // condition bits and factors are uniform loads (n_jobs == 0: one row of threads for otab)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per_slot = (int64_t)(n_jobs > 0 ? n_jobs : 1) << tiles_log;
    if (i >= (int64_t)S * per_slot) return;
    const int slot = (int)(i / per_slot);
    const int64_t rem = i - (int64_t)slot * per_slot;
    const int j = (int)(rem >> tiles_log);
    uint64_t t = (uint64_t)rem & ((1ull << tiles_log) - 1ull);
    const uint64_t tile = t;
    if (dyn) fixed_bits = (uint64_t)dyn->init & classical;
    uint64_t outer = fixed_bits, m = walk;
    while (m) {
        const uint64_t low = m & (~m + 1ull);
        if (t & 1ull) outer |= low;
        t >>= 1;
        m ^= low;
    }
    if (slot == 0 && j == 0) otab[tile] = outer;
    if (n_jobs == 0) return;
    const OuterJob jb = jobs[j];
    const cxf<R> *rec = rec_all + (size_t)slot * rec_size;
    cxf<R> w = {(R)1, (R)0};
    for (int k = 0; k < jb.n; ++k)
        if ((outer >> obits[jb.bits_off + k]) & 1ull) w = mul(w, rec[jb.rec_off + k]);
    wtab[(((int64_t)slot << tiles_log) + (int64_t)tile) * n_jobs + j] = w;
}

// A stage's sheared amplitudes exceed the state's by up to the inverse of its factors' product:
// 2^60 stays far inside the float range, and 48 noise-free Hadamards take 2^24 of it.
constexpr double kShearMin = 0x1p-60;

// One thread per (slot, op), then one wave per (slot, stage) for the products of the stages' factors
// alpha, for the slots slot_base, ..., slot_base + slots - 1 of S.  blockIdx.y: the pass, pass0 + blockIdx.y
// of the program, with its own record area; a launch per pass took 5 us of a chain of loads for 0.2 ms
// passes (Grover n = 20), the same as one for 32.
// Few threads, each with a chain of loads and products: the descriptors are read together, and no bound on
// the workgroup is given, with which the compiler moves the factors from scratch memory to the LDS (QFT
// n = 8, complex<float>, 3001 slots: 24.6 us with a bound of 128 threads, 16.0 without).
template <typename R>
__global__ void k_pass_prep(int S, int slot_base, int slots, int pass0, ProgramDev prog, const double *tab,
                            const qs_gate *gates, char *rec_base, uint64_t basis, const RunParams *dyn, PassAreas ar)
{
    const PassDesc *pd = prog.passes + pass0 + blockIdx.y;
    const int expand = pd->expand, op_begin = pd->op_begin, n_ops = pd->op_end - op_begin, rec_size = pd->rec_size;
    const int threads_log = pd->K - pd->RB;
    const int stage_begin = pd->stage_begin, n_stages = pd->stage_end - stage_begin;
    const int op_blocks = (int)(((int64_t)n_ops * slots + 127) / 128);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const OpDesc op = prog.ops[i < (int64_t)n_ops * slots ? op_begin + (int)(i % n_ops) : 0];
    if (expand) return;   // (launch_expand_prep)
    cxf<R> *rec_all = reinterpret_cast<cxf<R> *>(rec_base + blockIdx.y * ar.rec_stride);
    if ((int)blockIdx.x >= op_blocks) {
        const int64_t w = (int64_t)((int)blockIdx.x - op_blocks) * 2 + (threadIdx.x >> 6);
        if (w >= (int64_t)slots * n_stages) return;
        const int slot = (int)(w / n_stages), lane = (int)(threadIdx.x & 63u);
        const StageDesc sd = prog.stages[stage_begin + (int)(w % n_stages)];
        if (sd.scale_rec < 0) return;
        double f = 1.0;
        for (int oi = sd.op_begin + lane; oi < sd.op_end; oi += 64) {
            const OpDesc &op = prog.ops[oi];
            if (!(op.flags & OPF_SHEAR)) continue;
            f *= tab[((uint64_t)op.gate * S + slot_base + slot) * 8];
        }
        for (int off = 32; off > 0; off >>= 1) f *= __shfl_xor(f, off, 64);
        // too small a product (or NaN): the stage runs the matrices themselves, the entry is (1, 0)
        const bool sheared = fabs(f) >= kShearMin;
        if (lane == 0)
            rec_all[(size_t)slot * rec_size + sd.scale_rec] = sheared ? cxf<R>{(R)f, (R)1} : cxf<R>{(R)1, (R)0};
        return;
    }
    if (i >= (int64_t)n_ops * slots) return;
    if (dyn) basis = dyn->init;
    const int slot = (int)(i / n_ops);
    cxf<R> *blk = rec_all + (size_t)slot * rec_size;
    cxf<R> *rec = blk + op.rec;
    auto tabc = [&](int g) {
        const double *t = tab + ((uint64_t)g * S + slot_base + slot) * 8;
        return make_double2(t[0], t[1]);
    };
    auto put = [&](cxf<R> *dst, double2 v) { *dst = cxf<R>{(R)v.x, (R)v.y}; };
    if (op.type == OP_U1) {
        const double *t = tab + ((uint64_t)op.gate * S + slot_base + slot) * 8;
        const bool chain = (op.flags & OPF_CHAIN) != 0;
        double2 uni = make_double2(1.0, 0.0);
        if (op.flags & OPF_SHEAR) {
            put(rec, make_double2(t[0], t[2] / t[0]));
            for (int k = 1; k < 4; ++k) put(rec + k, make_double2(t[2 * k], 0.0));
        } else if (chain) {
            // phase-chain layout: the real matrix in the even words, the input phase in words
            // 1 and 3; the phase joins the folded input block, else record entry 4
            for (int k = 0; k < 4; ++k) put(rec + k, make_double2(t[2 * k], 0.0));
            uni = make_double2(t[1], t[3]);
            if (op.flags & OPF_UPHASE) put(rec + 4, uni);
        } else {
            for (int k = 0; k < 4; ++k) put(rec + k, make_double2(t[2 * k], t[2 * k + 1]));
        }
        for (int post = 0; post < 2; ++post) {
            int block = post ? op.post_rec : op.pre_rec;
            if (block < 0) continue;
            double2 preg[kMaxRegBits], ptid[10];
            double2 ubas = make_double2(1.0, 0.0);     // the block's basis-conditioned factors
            for (int k = 0; k < kMaxRegBits; ++k) preg[k] = make_double2(1.0, 0.0);
            for (int k = 0; k < 10; ++k) ptid[k] = make_double2(1.0, 0.0);
            for (int k = op.pref_begin; k < op.pref_end; ++k) {
                const PrepRef pr = prog.prefs[k];
                if (pr.post != post) continue;
                double2 ph = tabc(pr.gate);
                if (pr.kind == PR_REG) preg[pr.bit] = dmul(preg[pr.bit], ph);
                else if (pr.kind == PR_THREAD) ptid[pr.bit] = dmul(ptid[pr.bit], ph);
                else if (pr.kind == PR_BASIS) {
                    if ((basis >> pr.bit) & 1ull) ubas = dmul(ubas, ph);
                } else put(blk + pr.slot_entry, ph);
            }
            cxf<R> *b = blk + block;
            for (int k = 0; k < 4; ++k) put(b + k, k < kMaxRegBits ? preg[k] : make_double2(1.0, 0.0));
            for (int x = 0; x < 32; ++x) {
                double2 w = dmul(ubas, post ? make_double2(1.0, 0.0) : uni);
                for (int k = 0; k < 5; ++k)
                    if ((x >> k) & 1) w = dmul(w, ptid[k]);
                put(b + 4 + x, w);
            }
            for (int y = 0; y < 16; ++y) {
                double2 w = make_double2(1.0, 0.0);
                for (int k = 0; k < 4; ++k)
                    if ((y >> k) & 1) w = dmul(w, ptid[5 + k]);
                put(b + 36 + y, w);
            }
            if (threads_log > 9) {
                put(b + 52, make_double2(1.0, 0.0));
                put(b + 53, ptid[9]);
            }
        }
    } else if (op.type == OP_U2) {
        const double *m = gates[op.gate].m;
        for (int k = 0; k < 16; ++k) put(rec + k, make_double2(m[2 * k], m[2 * k + 1]));
    } else {
        put(rec, op.diag_kind == DIAG_PHASE ? tabc(op.gate) : make_double2(-1.0, 0.0));
    }
}

// Record entries per stage: 8 KiB of records (a stage bounds the descriptor ranges the kernel
// walks between two plan boundaries); 0 when the tile does not fit the 160 KiB of LDS.
int stage_rec_cap(qs_dtype dt, int K)
{
    const size_t cxs = dt == QS_C64 ? 8 : 16;
    if ((size_t(1) << K) * cxs > 160 * 1024) return 0;
    return (int)(8192 / cxs);
}

// LDS of one block: its tile.
size_t fused_lds_bytes(qs_dtype dt, int K)
{
    return (size_t(1) << K) * (dt == QS_C64 ? 8 : 16);
}

hipError_t launch_pass_prep(qs_dtype dt, int S, int slot_base, int slots, const PassDesc *h, int count, int pass0,
                            ProgramDev prog, const double *tab, const qs_gate *gates_dev, void *rec, const PassAreas &ar,
                            int64_t basis, const RunParams *dyn, hipStream_t st)
{
    uint64_t blocks = 0, entries = 0;
    for (int p = 0; p < count; ++p) {
        const uint64_t tot = (uint64_t)(h[p].op_end - h[p].op_begin) * slots;
        if (tot == 0 || h[p].expand) continue;
        blocks = std::max(blocks, (tot + 127) / 128 + ((uint64_t)slots * (h[p].stage_end - h[p].stage_begin) + 1) / 2);
        entries += (uint64_t)h[p].rec_size;
    }
    if (blocks == 0) return hipSuccess;
    TimedLaunch tl("prep", (double)slots * entries * (dt == QS_C64 ? 8 : 16), st);
    const dim3 grid((unsigned)blocks, (unsigned)count);
    if (dt == QS_C64)
        hipLaunchKernelGGL(k_pass_prep<float>, grid, dim3(128), 0, st, S, slot_base, slots, pass0, prog, tab, gates_dev,
                           (char *)rec, (uint64_t)basis, dyn, ar);
    else
        hipLaunchKernelGGL(k_pass_prep<double>, grid, dim3(128), 0, st, S, slot_base, slots, pass0, prog, tab, gates_dev,
                           (char *)rec, (uint64_t)basis, dyn, ar);
    return hipGetLastError();
}

hipError_t launch_block_prep(qs_dtype dt, int S, const PassDesc *h, ProgramDev prog, void *rec, hipStream_t st)
{
    const int n_rounds = h->round_end - h->round_begin;
    const int64_t tot = (int64_t)S * n_rounds * 16;
    if (tot == 0 || dt != QS_C64) return hipSuccess;
    TimedLaunch tl("prep", (double)S * n_rounds * kBlockRecEntries * 8.0, st);
    hipLaunchKernelGGL(k_block_prep<float>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, S, h->round_begin,
                       n_rounds, h->rec_size, prog, (cxf<float> *)rec);
    return hipGetLastError();
}

hipError_t launch_pass_jobs(qs_dtype dt, int S, const PassDesc *h, int count, int pass0, ProgramDev prog,
                            const void *rec, void *wt, const PassAreas &ar, int64_t init, int64_t basis,
                            const RunParams *dyn, hipStream_t st)
{
    uint64_t blocks = 0, products = 0;
    for (int p = 0; p < count; ++p) {
        const int n_jobs = h[p].job_end - h[p].job_begin;
        const bool fill = pass0 + p == 0 && init >= 0 && h[p].zero_fill;
        const uint64_t tiles = (uint64_t)S
                               << __builtin_popcountll(fill ? h[p].outer_mask : h[p].outer_mask & ~h[p].classical);
        blocks = std::max(blocks, (tiles * (n_jobs > 0 ? n_jobs : 1) + 255) / 256);
        products += tiles * n_jobs;
    }
    TimedLaunch tl("jobs", (double)products * (dt == QS_C64 ? 8 : 16), st);
    const dim3 grid((unsigned)blocks, (unsigned)count);
    if (dt == QS_C64)
        hipLaunchKernelGGL(k_pass_jobs<float>, grid, dim3(256), 0, st, S, pass0, init >= 0 ? 1 : 0, (uint64_t)basis,
                           prog.passes, prog.jobs, prog.obits, (const char *)rec, dyn, (char *)wt, ar);
    else
        hipLaunchKernelGGL(k_pass_jobs<double>, grid, dim3(256), 0, st, S, pass0, init >= 0 ? 1 : 0, (uint64_t)basis,
                           prog.passes, prog.jobs, prog.obits, (const char *)rec, dyn, (char *)wt, ar);
    return hipGetLastError();
}

hipError_t fused_prepare_attributes()
{
    const hipError_t e = fused_attributes<float>();
    return e != hipSuccess ? e : fused_attributes<double>();
}

int fused_walked_bits(int n, const PassDesc *pass_host, int64_t init)
{
    const bool fill = init >= 0 && pass_host->zero_fill;
    return n - pass_host->K - (fill ? 0 : __builtin_popcountll(pass_host->classical));
}

hipError_t launch_fused_pass(void *psi, qs_dtype dt, int n, int S, const PassDesc *pass_host,
                             int pass_index, int64_t init, int64_t basis, ProgramDev prog, const void *rec,
                             const void *wtab, const uint64_t *otab, hipStream_t st, const RunParams *dyn,
                             double *ovl, int slot_base, int slots)
{
    const PassDesc &h = *pass_host;
    if (h.state) return hipErrorInvalidValue;   // launch_state_pass
    if (h.expand)
        return launch_expand_pass(psi, dt, n, S, pass_host, pass_index, init, basis, prog, rec, wtab, otab, st, dyn, ovl,
                                  slot_base, slots);
    size_t lds = fused_lds_bytes(dt, h.K);
    const int rec_cap = stage_rec_cap(dt, h.K);
    if (lds > 160 * 1024 || rec_cap <= 0 || basis < 0) return hipErrorInvalidValue;
    if (ovl && (slots < 1 || slot_base < 0 || slot_base + slots > S)) return hipErrorInvalidValue;
    const int S_run = ovl ? slots : S;
    // Algorithmic bytes: a pass writes the tiles that can hold amplitude (a 2^-popcount(classical)
    // share; every tile when the first pass stores the zeros) and reads, except the first pass,
    // the amplitudes of the support inside them (a further 2^-popcount(lclassical) share).
    const bool fill_all = init >= 0 && h.zero_fill;
    const double tiles_share = fill_all ? 1.0 : std::ldexp(1.0, -__builtin_popcountll(h.classical));
    const double read_share = init >= 0 ? 0.0 : std::ldexp(1.0, -__builtin_popcount(h.lclassical));
    // with the overlaps: slot 0's tiles once more (read from HBM once, by the first slot of a tile)
    const double ref_share = ovl && slot_base > 0 ? 1.0 : 0.0;
    TimedLaunch tl("fused",
                   ((1.0 + read_share) * (double)S_run + ref_share) * tiles_share * std::ldexp(1.0, n) * amp_bytes(dt),
                   st);
    if (dt == QS_C64)
        return fused_launch((float *)psi, n, S, h, pass_index, rec_cap, init, basis, dyn, prog, rec, wtab, otab, lds, st,
                            ovl, slot_base, slots);
    return fused_launch((double *)psi, n, S, h, pass_index, rec_cap, init, basis, dyn, prog, rec, wtab, otab, lds, st, ovl,
                        slot_base, slots);
}

}  // namespace qs
