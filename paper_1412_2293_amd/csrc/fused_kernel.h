// Fused pass kernel: a run of gates whose non-diagonal targets lie in one set of K "tile"
// qubits is applied to every tile of 2^K amplitudes in a single read and write of HBM.
//
// Layout: tile-local index bit j is physical bit q_pos[j]; the other n - K bits number the
// tiles (one workgroup per tile and slot).  Each thread keeps 2^RB amplitudes in registers.
// A round names the RB tile-local bits held in registers; a one-qubit gate on one of them
// updates register pairs (Section 2's amplitude-pair update), a two-qubit gate register
// quadruples.  Between rounds the tile is re-distributed through LDS.  Controlled phases and
// sign flips are diagonal: a controlled phase is folded into the neighbouring one-qubit gate
// on one of its qubits as a phase on that gate's |1> input or output, conditioned on the other
// qubit, which is a tile-constant, thread-constant or register bit here.
#pragma once

#include <cmath>
#include <type_traits>

#include "cplx.h"
#include "internal.h"
#include "regops.h"

namespace qs {


__device__ __forceinline__ uint32_t swz(uint32_t l)
{
    return lds_swizzle(l);
}

template <int RB>
__device__ __forceinline__ void reg_offsets(uint32_t reg_mask, int K, uint32_t (&roff)[1 << RB])
{
    uint32_t pos[RB];
    int b = 0;
    for (int j = 0; j < K && b < RB; ++j)
        if (reg_mask & (1u << j)) pos[b++] = 1u << j;
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
        uint32_t o = 0;
#pragma unroll
        for (int k = 0; k < RB; ++k)
            if (r & (1 << k)) o |= pos[k];
        roff[r] = o;
    }
}

// ---------------------------------------------------------------------------------------
// Dense 16 x 16 blocks on the FP32 matrix cores (rounds the planner marks with a block record).
// In a round the 16 registers of a thread are the 16 states of the round's four qubits (register
// index = block index) and the thread id numbers the columns.  A 16 x 16 x 4 product takes its
// K index from lane bits 4, 5 and a chunk index, so register bits 0, 1 are first exchanged with
// lane bits 4, 5 (one lane-half swap per register pair and component); then register
// g + 4c of lane group j holds block state j + 4c of column group g.  With the block as the real
// 32 x 32 matrix [[Re U, -Im U], [Im U, Re U]] acting on [Re x; Im x], eight products of four
// rows each give the real and imaginary output rows of one column group.  Output register i of
// lane group j holds row 4j + i; it is stored at register g + 4i, and after the exchange back
// the register index is j + 4i.  The operand table holds the block with its rows permuted by
// P(4j + i) = 4i + j, so that register j + 4i ends with output state j + 4i.
// ---------------------------------------------------------------------------------------
typedef float mf4 __attribute__((ext_vector_type(4)));

// (lo, hi): the same register pair of a lane half; exchange the upper 16 lanes of each 32 of lo
// with the lower 16 of hi (a transpose of register bit and lane bit 4).
__device__ __forceinline__ void lane_swap16(tv<float> &lo, tv<float> &hi)
{
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo.x), __float_as_uint(hi.x), false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo.y), __float_as_uint(hi.y), false, false);
    lo = tv<float>{__uint_as_float(x[0]), __uint_as_float(y[0])};
    hi = tv<float>{__uint_as_float(x[1]), __uint_as_float(y[1])};
}

// The same for lane bit 5 (upper 32 lanes of lo with the lower 32 of hi).
__device__ __forceinline__ void lane_swap32(tv<float> &lo, tv<float> &hi)
{
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo.x), __float_as_uint(hi.x), false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo.y), __float_as_uint(hi.y), false, false);
    lo = tv<float>{__uint_as_float(x[0]), __uint_as_float(y[0])};
    hi = tv<float>{__uint_as_float(x[1]), __uint_as_float(y[1])};
}

__device__ __forceinline__ void swap_reg01_lane45(tv<float> (&a)[16])
{
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (!(r & 1)) lane_swap16(a[r], a[r | 1]);
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (!(r & 2)) lane_swap32(a[r], a[r | 2]);
}

// y = U x for every column of the register tile (64 products); tab: this lane's 16 operand
// values, entry ob * 8 + c = row block ob (real, imaginary outputs) and K chunk c (rows 4c..4c+3
// of [Re x; Im x]).
__device__ __forceinline__ void block_apply(tv<float> (&a)[16], const float (&A)[16])
{
    swap_reg01_lane45(a);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        mf4 re = {0.f, 0.f, 0.f, 0.f}, im = re;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            re = __builtin_amdgcn_mfma_f32_16x16x4f32(A[c], a[g + 4 * c].x, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f32_16x16x4f32(A[8 + c], a[g + 4 * c].x, im, 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            re = __builtin_amdgcn_mfma_f32_16x16x4f32(A[4 + c], a[g + 4 * c].y, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f32_16x16x4f32(A[12 + c], a[g + 4 * c].y, im, 0, 0, 0);
        }
        // column group g's inputs are consumed: its outputs take their registers
#pragma unroll
        for (int i = 0; i < 4; ++i) a[g + 4 * i] = tv<float>{re[i], im[i]};
    }
    swap_reg01_lane45(a);
}

// a[r] *= w for the registers whose bit P is set (a phase on the |1> state of register bit P).
template <typename R, int RB, int P>
__device__ __forceinline__ void phase_on_bit(tv<R> (&a)[1 << RB], cxf<R> w)
{
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r)
        if ((r >> P) & 1) a[r] = tvec(mul(w, cx<R>(a[r])));
}

template <typename R, int RB>
__device__ __forceinline__ void dispatch_phase_on_bit(int p, tv<R> (&a)[1 << RB], cxf<R> w)
{
    if (RB > 1 && p == 0) phase_on_bit<R, RB, 0>(a, w);
    else if (RB > 2 && p == 1) phase_on_bit<R, RB, 1 % RB>(a, w);
    else if (RB > 3 && p == 2) phase_on_bit<R, RB, 2 % RB>(a, w);
    else phase_on_bit<R, RB, RB - 1>(a, w);
}

// LDS of one block: the tile only.  Op and round descriptors, matrices and register-bit phase
// factors are read with scalar loads; the per-thread phase tables of a folded block with vector
// loads of the slot's records (a few KB, cache resident); the per-tile products of the phases
// conditioned on tile-number bits come from the table written by k_pass_jobs.

// Register tiles of 16 complex<float> or 8 complex<double> (and more) need more than 128
// VGPRs: those tiles have at most 256 threads and may use the whole register file.
template <typename R, int RB>
constexpr bool kWideTile = RB == 4 || (sizeof(R) == 8 && RB == 3);

// Waves per SIMD the register allocation must allow.  complex<float> with 16-register tiles is
// held to 128 VGPRs, so that four 256-thread blocks share a CU (their 32 KiB tiles fit the
// 160 KiB of LDS): more waves hide the tile loads and the LDS exchanges better than the
// registers the compiler would otherwise keep for scheduling.
template <typename R, int RB>
constexpr int kMinWaves = (sizeof(R) == 4 && RB == 4) ? 4 : 1;

// UNI: whether blocks whose factors do not depend on thread-id bits take their per-thread factor
// with a uniform load (the host picks this variant for passes where most blocks are such; the
// other keeps the per-thread lookups branch-free, which schedules better when few are).
// ZV: which one-qubit ops act on a target that still holds its basis bit (the zero-input
// updates): 0 none, 1 some, 2 all.  Variants 0 and 2 leave out the code paths they cannot take
// (the op dispatch of variant 1 is the largest; without it random layers measured 2-3% faster).
// ZV 3: as 2, and every one-qubit op has a real matrix, no input phase and at most a uniform
// output factor (the QFT's passes), so the op loop holds only those paths.  ZV 4: as 0, and
// every one-qubit op has a real matrix and no folded phase.  ZV 6: as 4, and every one-qubit op is
// a sheared reflection (Grover's Hadamard layers).  ZV 5:
// no one-qubit op at all (density-matrix passes of dense two-qubit superoperators and diagonal
// patterns).  ZV 7: as 5, with the diagonal ops' products collected.
// MIX: whether the pass has ops other than one-qubit gates (dense two-qubit gates, diagonal
// patterns left standalone); without them the op loop holds only the one-qubit paths (QFT
// and random-layer passes 1-2% faster).
template <typename R, int RB, bool UNI, bool BLK, int ZV, bool MIX>
__global__ void __launch_bounds__((kWideTile<R, RB>) ? 256 : 512)
    __attribute__((amdgpu_waves_per_eu(kMinWaves<R, RB>, 8))) k_fused(R *__restrict__ psi, int n, int S, int pass_index,
                                                  int rec_cap, int64_t init, int64_t basis, uint32_t blocal,
                                                  const RunParams *__restrict__ dyn,
                                                  const PassDesc *__restrict__ g_passes,
                                                  const StageDesc *__restrict__ g_stages,
                                                  const RoundDesc *__restrict__ g_rounds,
                                                  const OpDesc *__restrict__ g_ops,
                                                  const cxf<R> *__restrict__ rec_all,
                                                  const cxf<R> *__restrict__ wtab,
                                                  const uint64_t *__restrict__ otab,
                                                  double *__restrict__ ovl, int slot_base, int slots)
{
    // Descriptor arrays as separate read-only, non-aliasing arguments: their uniform reads
    // become scalar loads that do not wait on the tile's vector memory traffic.
    struct {
        const PassDesc *__restrict__ passes;
        const StageDesc *__restrict__ stages;
        const RoundDesc *__restrict__ rounds;
        const OpDesc *__restrict__ ops;
    } prog = {g_passes, g_stages, g_rounds, g_ops};
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NR = 1 << RB;
    const PassDesc *pd = prog.passes + pass_index;
    const int K = pd->K;
    // A run starts in the basis state |basis>, and a physical qubit no non-diagonal gate has
    // touched still holds its basis value (controlled phases only rescale), so only the tiles
    // that agree with it on the pass's classical bits hold amplitude, and inside a tile only the
    // amplitudes that agree with it on the tile-local classical bits.  A pass is launched over
    // the tiles that hold amplitude (its blocks walk the other tile-number bits) and reads only
    // those amplitudes; the first pass also stores the other tiles as zeros when no later pass
    // rewrites them.
    const bool first = init >= 0;
    if (dyn) {
        basis = dyn->init;
        if (first) init = basis;
    }
    const bool fill = first && pd->zero_fill;
    const uint64_t walk = fill ? pd->outer_mask : (pd->outer_mask & ~pd->classical);
    const int tiles_log = __builtin_popcountll(walk);
    // Block order: slot-major, so that the blocks in flight share one slot's records.  When the
    // pass also forms the overlaps with slot 0 (slots [slot_base, slot_base + slots)), tile-major
    // with the slot fastest: all slots of a tile run together and read slot 0's tile from the
    // caches.  (Measured against groups of 2^10 tiles, group-major, and against slot groups of 8
    // with one slot per XCD: both slower, as slot 0's tiles are then reused from further away.)
    int slot;
    uint64_t tile;
    if (ovl) {
        slot = slot_base + (int)(blockIdx.x % (unsigned)slots);
        tile = blockIdx.x / (unsigned)slots;
    } else {
        slot = (int)(blockIdx.x >> tiles_log);
        tile = (uint64_t)blockIdx.x & ((1ull << tiles_log) - 1ull);
    }
    // uniform by construction; the division above runs on the vector ALUs, so say so, and the
    // record and table pointers derived from them stay in scalar registers
    slot = __builtin_amdgcn_readfirstlane(slot);
    tile = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(tile >> 32)) << 32) |
           (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)tile);
    const uint64_t bidx = ((uint64_t)slot << tiles_log) | tile;
    const uint32_t tid = threadIdx.x, nthr = blockDim.x;
    const cxf<R> *__restrict__ rec = rec_all + (size_t)slot * pd->rec_size;
    // this tile's products of the phases conditioned on tile-number bits (one per outer job)
    const cxf<R> *__restrict__ wout = wtab + bidx * (size_t)(pd->job_end - pd->job_begin);

    // Outer (tile-number) bits of the physical index, written for this launch by k_pass_jobs.
    const uint64_t outer = otab[tile];
    // Load (and store) layout: the register bits are the tile-local bits of its round
    // descriptor's mask, the thread id fills the others, lowest first.  lthr0: the thread's
    // tile-local index bits in that layout (a zero bit inserted at each register bit).
    const uint32_t load_mask = prog.rounds[pd->load_round].reg_mask;
    uint64_t gthr = outer;
    uint32_t lthr0 = tid;
    {
        uint32_t m = load_mask;
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const uint32_t b = (uint32_t)__builtin_ctz(m);
            const uint32_t lo = lthr0 & ((1u << b) - 1u);
            lthr0 = ((lthr0 ^ lo) << 1) | lo;
            m &= m - 1u;
        }
        for (int j = 0; j < K; ++j)
            if ((lthr0 >> j) & 1u) gthr |= 1ull << pd->q_pos[j];
    }
    uint64_t greg[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) greg[r] = pd->reg_off[r];
    R *base = psi + ((uint64_t)slot << (n + 1));
    // the basis index's bits at the tile-local positions (from the host, or here when the
    // basis comes from the device block)
    if (dyn) {
        blocal = 0;
        for (int j = 0; j < K; ++j)
            if (((uint64_t)basis >> pd->q_pos[j]) & 1ull) blocal |= 1u << j;
    }
    tv<R> a[NR];
    if (fill && ((outer ^ (uint64_t)basis) & pd->classical) != 0) {
        // a tile of the first pass outside the support: zeros (uniform per block)
#pragma unroll
        for (int r = 0; r < NR; ++r)
            __builtin_nontemporal_store(tv<R>{(R)0, (R)0}, reinterpret_cast<tv<R> *>(base + 2 * (gthr | greg[r])));
        if (ovl && tid < 3) ovl[bidx * 3 + tid] = 0.0;
        return;
    }
    if (init >= 0) {
        // first pass of a run: every slot starts in the basis state |init>, made here
        // instead of read from memory
#pragma unroll
        for (int r = 0; r < NR; ++r) a[r] = tv<R>{(gthr | greg[r]) == (uint64_t)init ? (R)1 : (R)0, (R)0};
    } else {
        // read only the amplitudes that can be nonzero: tile-local index lthr0 | roff[r] agrees
        // with the basis index on the tile-local classical bits (thread part per lane, register
        // part uniform)
        const uint32_t lc = pd->lclassical;
        if (lc == 0) {
#pragma unroll
            for (int r = 0; r < NR; ++r)
                a[r] = __builtin_nontemporal_load(reinterpret_cast<const tv<R> *>(base + 2 * (gthr | greg[r])));
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) a[r] = tv<R>{(R)0, (R)0};
            // only lanes whose thread part agrees with the basis read anything, so a wave with
            // none of them (most waves when few tile bits are touched) skips the loads
            const bool tok = ((lthr0 ^ blocal) & lc & ~load_mask) == 0;
            if (tok) {
                const RoundDesc *ld = prog.rounds + pd->load_round;
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const bool rok = ((ld->roff[r] ^ blocal) & lc & load_mask) == 0;
                    if (rok) {
                        const uint64_t i = gthr | greg[r];
                        a[r] = __builtin_nontemporal_load(reinterpret_cast<const tv<R> *>(base + 2 * i));
                    }
                }
            }
        }
    }

    // Register layout: tile-local index of register r of this thread = lthr | roff[r], with
    // roff from the current round's descriptor (cur_ri; at first the load layout's).  LDS addresses: swz(lthr | roff[r]) = swz(lthr) ^ swz(roff[r]); the register
    // part is the descriptor's sroff (one scalar load of 16 words), so each access costs one
    // XOR.  The tile sits at the start of the dynamic LDS, addressed directly.
    constexpr uint32_t CXS = sizeof(cxf<R>);
    typedef R v2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) v2 lds_v2;
    // the kernel declares no static LDS (checked on the host before its first launch), so the
    // dynamic LDS, and the tile at its start, begins at LDS address 0
    auto lds_put = [](uint32_t byte, cxf<R> x) {
        *reinterpret_cast<lds_v2 *>((size_t)byte) = v2{x.re, x.im};
    };
    auto lds_get = [](uint32_t byte) {
        const v2 v = *reinterpret_cast<const lds_v2 *>((size_t)byte);
        return cxf<R>{v.x, v.y};
    };
    uint32_t cur = load_mask;
    // current register layout as an index into the rounds array: loads through the kernel
    // argument with a uniform index stay scalar
    int cur_ri = pd->load_round;
    uint32_t lthr = lthr0;

    auto exchange_to = [&](uint32_t to, int ri) {
        __syncthreads();
        {
            // opaque to the optimiser, which would otherwise distribute the swizzle and the
            // scaling over every access (three VALU ops per access instead of one XOR)
            uint32_t sw = swz(lthr) * CXS;
            asm volatile("" : "+v"(sw));
            const RoundDesc *from = prog.rounds + cur_ri;
#pragma unroll
            for (int r = 0; r < NR; ++r) lds_put(sw ^ (from->sroff[r] * CXS), cx<R>(a[r]));
        }
        __syncthreads();
        const RoundDesc *rd = prog.rounds + ri;
        cur = to;
        cur_ri = ri;
        // the thread id deposited into the tile-local bits outside the registers: a zero bit
        // inserted at each register bit, lowest first (arithmetic, no table load to wait on)
        {
            uint32_t x = tid, m = to;
#pragma unroll
            for (int k = 0; k < RB; ++k) {
                const uint32_t b = (uint32_t)__builtin_ctz(m);
                const uint32_t lo = x & ((1u << b) - 1u);
                x = ((x ^ lo) << 1) | lo;
                m &= m - 1u;
            }
            lthr = x;
        }
        uint32_t sw = swz(lthr) * CXS;
        asm volatile("" : "+v"(sw));
#pragma unroll
        for (int r = 0; r < NR; ++r) a[r] = tvec(lds_get(sw ^ (rd->sroff[r] * CXS)));
    };

    // A diagonal-pattern op: its tile-local condition splits into the lane's thread bits (one
    // compare per lane) and the register bits (the same for every lane), so only the registers
    // whose bits match are multiplied (a Grover sign flip on all qubits touches one of 16).
    auto diag_op = [&](const OpDesc *op) {
        const bool ohit = (outer & op->omask) == op->ovalue;
        const uint32_t lmask = op->lmask, lvalue = op->lvalue;
        const uint32_t rm = prog.rounds[cur_ri].reg_mask;
        const bool thit = ohit && (lthr & lmask) == (lvalue & ~rm);
        const uint32_t rmask = lmask & rm, rval = lvalue & rm;
        const cxf<R> f = rec[op->rec];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if ((prog.rounds[cur_ri].roff[r] & rmask) == rval) {
                const tv<R> y = tvec(mul(f, cx<R>(a[r])));
                a[r] = thit ? y : a[r];
            }
        }
    };

    // ZV 7 (density matrices: many averaged phases between few superoperators): a diagonal op on one or
    // two register bits only multiplies its factor into the thread's product for those bits, and the
    // products reach the registers before the next dense op or exchange.  Applied one by one, each op
    // passed over half or a quarter of the registers, with a test per register (density matrix of the
    // 12-qubit QFT, 198 such ops in three passes: complex<float>, 282 us in the passes one by one, 195 with
    // the products; complex<double>, 330 and 287).  The products are held at twice the precision: in the
    // type's own they took 189 and 250 us, but equal layers of such ops came out up to four times
    // further off than one by one.
    constexpr bool DEFER = ZV == 7;
    cxprod<R> dw1[RB], dw2;
    dw2.clear();
#pragma unroll
    for (int k = 0; k < RB; ++k) dw1[k] = dw2;
    uint32_t dirty = 0;          // bit k: dw1[k] holds factors; bit 8: dw2, for the register bits in dpair
    uint32_t dpair = 0;
    auto flush = [&]() {
        if (dirty == 0) return;
        auto single = [&](auto pc) {
            constexpr int P = decltype(pc)::value;
            if (P < RB && ((dirty >> P) & 1u)) {
                const cxf<R> hi = dw1[P % RB].hi(), lo = dw1[P % RB].lo();
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if ((r >> P) & 1) a[r] = mul2(hi, lo, a[r]);
                dw1[P % RB].clear();
            }
        };
        single(std::integral_constant<int, 0>{});
        single(std::integral_constant<int, 1>{});
        single(std::integral_constant<int, 2>{});
        single(std::integral_constant<int, 3>{});
        if (dirty & 256u) {
            const cxf<R> hi = dw2.hi(), lo = dw2.lo();
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (((uint32_t)r & dpair) == dpair) a[r] = mul2(hi, lo, a[r]);
            dw2.clear();
        }
        dirty = 0;
    };
    // w: the thread's factor on register bit p0, or on p0 and p1
    auto collect = [&](int p0, int p1, cxf<R> w) {
        if (p1 >= 0) {
            const uint32_t pair = 1u << p0 | 1u << p1;
            if ((dirty & 256u) && pair != dpair) flush();
            dpair = pair;
            dirty |= 256u;
            dw2.times(w);
            return;
        }
        dirty |= 1u << p0;
        if (p0 == 0) dw1[0].times(w);
        else if (RB > 1 && p0 == 1) dw1[1 % RB].times(w);
        else if (RB > 2 && p0 == 2) dw1[2 % RB].times(w);
        else dw1[RB - 1].times(w);
    };
    // The diagonal ops from oi on, up to the next dense op or the round's end: their descriptors and
    // factors four at a time, so that four ops wait on two scalar loads in turn instead of eight.
    auto diag_run = [&](int oi, int oe) {
        const uint32_t rm = prog.rounds[cur_ri].reg_mask;
        for (;;) {
            constexpr int B = 4;
            int type[B], p0[B], p1[B], at[B];
            uint32_t lm[B], lv[B], cr[B];
            uint64_t om[B], ov[B];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const OpDesc *op = prog.ops + (oi + k < oe ? oi + k : oe - 1);
                type[k] = op->type;
                p0[k] = op->p0;
                p1[k] = op->p1;
                at[k] = op->rec;
                lm[k] = op->lmask;
                lv[k] = op->lvalue;
                cr[k] = op->creg;
                om[k] = op->omask;
                ov[k] = op->ovalue;
            }
            cxf<R> f[B];
#pragma unroll
            for (int k = 0; k < B; ++k) f[k] = rec[at[k]];
#pragma unroll
            for (int k = 0; k < B; ++k) {
                if (oi >= oe || type[k] == OP_U2) return oi;
                ++oi;
                if ((outer & om[k]) != ov[k]) continue;
                const bool hit = (lthr & lm[k]) == (lv[k] & ~rm);
                const cxf<R> w = {hit ? f[k].re : (R)1, hit ? f[k].im : (R)0};
                if (p0[k] >= 0) {
                    collect(p0[k], p1[k], w);
                } else if (cr[k]) {
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        if (((uint32_t)r & cr[k]) == cr[k]) a[r] = tvec(mul(w, cx<R>(a[r])));
                } else {
                    diag_op(prog.ops + oi - 1);
                }
            }
        }
    };

    for (int si = pd->stage_begin; si < pd->stage_end; ++si) {
        const StageDesc sd = prog.stages[si];
        bool sheared = false;   // the stage's one-qubit ops leave out their factors
        if constexpr (ZV == 6)
            if (sd.scale_rec >= 0) sheared = rec[sd.scale_rec].im != (R)0;
        for (int ri = sd.round_begin; ri < sd.round_end; ++ri) {
            const RoundDesc *rd = prog.rounds + ri;
            const uint32_t mask = rd->reg_mask;
            if (mask != cur) exchange_to(mask, ri);
            if constexpr (BLK && sizeof(R) == 4 && RB == 4) {
                // every round of a block pass is a block (the planner makes it all or none), so
                // this variant carries no op-by-op path
                {
                    // the round as one dense block: the ops' phases conditioned outside the
                    // registers before and after it (per op, on its target's |1> states)
                    const float *tp = reinterpret_cast<const float *>(rec + rd->block_rec) + (tid & 63u) * 16;
                    float A[16];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float4 q4 = *reinterpret_cast<const float4 *>(tp + 4 * k);
                        A[4 * k] = q4.x;
                        A[4 * k + 1] = q4.y;
                        A[4 * k + 2] = q4.z;
                        A[4 * k + 3] = q4.w;
                    }
                    for (int oi = rd->op_begin; oi < rd->op_end; ++oi) {
                        const OpDesc *op = prog.ops + oi;
                        const int flags = op->flags;
                        if (op->pre_rec >= 0 && (!(flags & OPF_PRE_UNI) || op->pre_job >= 0)) {
                            PhaseSet<R, RB> pre;
                            load_phases<R, RB>(pre, rec + op->pre_rec, rec + op->pre_rec, true, false,
                                               UNI && (flags & OPF_PRE_UNI) != 0, op->pre_job, wout, tid);
                            dispatch_phase_on_bit<R, RB>(op->p0, a, pre.w);
                        }
                    }
                    block_apply(a, A);
                    for (int oi = rd->op_begin; oi < rd->op_end; ++oi) {
                        const OpDesc *op = prog.ops + oi;
                        const int flags = op->flags;
                        if (op->post_rec >= 0 && (!(flags & OPF_POST_UNI) || op->post_job >= 0)) {
                            PhaseSet<R, RB> post;
                            load_phases<R, RB>(post, rec + op->post_rec, rec + op->post_rec, true, false,
                                               UNI && (flags & OPF_POST_UNI) != 0, op->post_job, wout, tid);
                            dispatch_phase_on_bit<R, RB>(op->p0, a, post.w);
                        }
                    }
                }
            } else {
            if constexpr (ZV == 3 && RB == 4) {
                // a round of untouched-target updates on register bits k-1, ..., 0: straight-line,
                // no per-op dispatch (its merges copy the register tile)
                const int seq = rd->seq;
                if (seq > 0) {
                    auto step = [&](int oi, auto pc) {
                        constexpr int PP = decltype(pc)::value;
                        const OpDesc *op = prog.ops + oi;
                        const cxf<R> *__restrict__ orec = rec + op->rec;
                        const int postr = op->post_rec, postj = op->post_job;
                        cxf<R> w = cxf<R>{(R)1, (R)0};
                        if (postr >= 0) {
                            w = rec[postr + 4];
                            if (postj >= 0) w = mul(w, wout[postj]);
                        }
                        const bool bit1 = (blocal & prog.rounds[cur_ri].roff[1 << PP]) != 0;
                        const R A = bit1 ? orec[1].re : orec[0].re;
                        const R Bm = bit1 ? orec[3].re : orec[2].re;
                        apply_u1_untouched<R, RB, PP>(a, A, cxf<R>{Bm * w.re, Bm * w.im});
                    };
                    const int ob = rd->op_begin;
                    if (seq == 4) {
                        step(ob, std::integral_constant<int, 3>{});
                        step(ob + 1, std::integral_constant<int, 2>{});
                        step(ob + 2, std::integral_constant<int, 1>{});
                        step(ob + 3, std::integral_constant<int, 0>{});
                    } else if (seq == 3) {
                        step(ob, std::integral_constant<int, 2>{});
                        step(ob + 1, std::integral_constant<int, 1>{});
                        step(ob + 2, std::integral_constant<int, 0>{});
                    } else if (seq == 2) {
                        step(ob, std::integral_constant<int, 1>{});
                        step(ob + 1, std::integral_constant<int, 0>{});
                    } else {
                        step(ob, std::integral_constant<int, 0>{});
                    }
                    continue;
                }
            }
            if constexpr ((ZV == 4 || ZV == 6) && RB == 4) {
                // rounds of real updates of touched targets on register bits 0, ..., k-1 in turn
                // (seq = k), or two such runs of four around one diagonal pattern (seq = 9):
                // straight-line, the target bits fixed at compile time
                const int seq = rd->seq;
                if (seq > 0) {
                    auto run = [&](auto sc) {
                        auto step = [&](int oi, auto pc) {
                            constexpr int PP = decltype(pc)::value;
                            const cxf<R> *__restrict__ orec = rec + prog.ops[oi].rec;
                            if constexpr (decltype(sc)::value) {
                                apply_u1_shear<R, RB, PP>(a, orec[0].im);
                            } else {
                                PhaseSet<R, RB> none;
                                none.any = false;
                                const cxf<R> m[4] = {orec[0], orec[1], orec[2], orec[3]};
                                apply_u1_real<R, RB, PP, 0, 0, 0>(a, m, none, none);
                            }
                        };
                        auto run4 = [&](int ob) {
                            step(ob, std::integral_constant<int, 0>{});
                            step(ob + 1, std::integral_constant<int, 1>{});
                            step(ob + 2, std::integral_constant<int, 2>{});
                            step(ob + 3, std::integral_constant<int, 3>{});
                        };
                        const int ob = rd->op_begin;
                        if (seq == 9) {
                            run4(ob);
                            diag_op(prog.ops + ob + 4);
                            run4(ob + 5);
                        } else if (seq == 4) {
                            run4(ob);
                        } else if (seq == 3) {
                            step(ob, std::integral_constant<int, 0>{});
                            step(ob + 1, std::integral_constant<int, 1>{});
                            step(ob + 2, std::integral_constant<int, 2>{});
                        } else if (seq == 2) {
                            step(ob, std::integral_constant<int, 0>{});
                            step(ob + 1, std::integral_constant<int, 1>{});
                        } else {
                            step(ob, std::integral_constant<int, 0>{});
                        }
                    };
                    if (ZV == 6 && sheared) run(std::true_type{});
                    else run(std::false_type{});
                    continue;
                }
            }
            const int oe = rd->op_end;
            for (int oi = rd->op_begin; oi < oe; ++oi) {
                if constexpr (DEFER) {
                    oi = diag_run(oi, oe);
                    if (oi >= oe) break;
                }
                const OpDesc *op = prog.ops + oi;
                const int type = DEFER ? (int)OP_U2 : op->type;
                const cxf<R> *__restrict__ orec = rec + op->rec;
                if (ZV == 6 && sheared && type == OP_U1) {
                    dispatch_u1_shear<R, RB>(op->p0, a, orec[0].im);
                } else if ((ZV == 4 || ZV == 6) && type == OP_U1) {
                    // every one-qubit op of the pass: real matrix, no folded phase, target
                    // already touched (the general pair update)
                    cxf<R> m[4] = {orec[0], orec[1], orec[2], orec[3]};
                    PhaseSet<R, RB> none;
                    none.any = false;
                    dispatch_u1_pp<R, RB, 0, 0, 0>(op->p0, true, a, m, none, none);
                } else if (ZV == 3 && type == OP_U1) {
                    // every one-qubit op of the pass: real matrix, target still untouched, no
                    // input phase, output phase at most one uniform factor
                    cxf<R> m[4] = {orec[0], orec[1], orec[2], orec[3]};
                    // an op without an output block takes the factor 1: one update path per
                    // target and input instead of two
                    PhaseSet<R, RB> pre, post;
                    pre.any = false;
                    post.any = true;
                    const int postr = op->post_rec, postj = op->post_job;
                    post.w = cxf<R>{(R)1, (R)0};
                    if (postr >= 0) {
                        post.w = rec[postr + 4];
                        if (postj >= 0) post.w = mul(post.w, wout[postj]);
                    }
                    const bool bit1 = (blocal & prog.rounds[cur_ri].roff[1 << op->p0]) != 0;
                    if (bit1) dispatch_u1_pp<R, RB, 0, 1, 2>(op->p0, true, a, m, pre, post);
                    else dispatch_u1_pp<R, RB, 0, 1, 1>(op->p0, true, a, m, pre, post);
                } else if (ZV != 5 && ZV != 7 && type == OP_U1) {
                    cxf<R> m[4] = {orec[0], orec[1], orec[2], orec[3]};
                    PhaseSet<R, RB> pre, post;
                    const int flags = op->flags;
                    const int prer = op->pre_rec, postr = op->post_rec;
                    const int prej = op->pre_job, postj = op->post_job;
                    // a target qubit no earlier gate has touched holds the basis bit: when that
                    // bit is 0 every |1> input is zero (and its input phase has nothing to do),
                    // when it is 1 every |0> input
                    const bool untouched = ZV >= 2 || (ZV == 1 && ((op->creg >> op->p0) & 1u) != 0);
                    const bool bit1 = (blocal & prog.rounds[cur_ri].roff[1 << op->p0]) != 0;
                    const bool zero_in = untouched && !bit1;
                    const int zin = untouched ? (bit1 ? 2 : 1) : 0;
                    int prekind;
                    if (zero_in) {
                        pre.any = false;
                        prekind = 0;
                    } else if (flags & OPF_UPHASE) {
                        // uniform input phase (an inner phase-chain member with no folded block)
                        pre.any = true;
                        pre.w = orec[4];
                        prekind = 1;
                    } else {
                        const bool bits = !(flags & OPF_PREW);
                        load_phases<R, RB>(pre, rec + prer, rec + prer, prer >= 0, bits,
                                           UNI && (flags & OPF_PRE_UNI) != 0, prej, wout, tid);
                        prekind = prer < 0 ? 0 : bits ? 2 : 1;
                    }
                    const bool postbits = !(flags & OPF_POSTW);
                    load_phases<R, RB>(post, rec + postr, rec + postr, postr >= 0, postbits,
                                       UNI && (flags & OPF_POST_UNI) != 0, postj, wout, tid);
                    const int postkind = postr < 0 ? 0 : postbits ? 2 : 1;
                    dispatch_u1<R, RB>(op->p0, (flags & OPF_REAL) != 0, prekind, zin, postkind, a, m, pre,
                                       post);
                } else if (MIX && type == OP_U2) {
                    if constexpr (DEFER) flush();
                    cxf<R> m[16];
#pragma unroll
                    for (int k = 0; k < 16; ++k) m[k] = orec[k];
                    dispatch_u2<R, RB>(op->p0, op->p1, (op->flags & OPF_REAL) != 0, a, m);
                } else if (MIX) {
                    diag_op(op);
                }
            }
            if constexpr (DEFER) flush();
            }
        }
        if constexpr (ZV == 6)
            if (sheared) {
                const R f = rec[sd.scale_rec].re;
#pragma unroll
                for (int r = 0; r < NR; ++r) a[r] *= f;
            }
    }
    // Slot 0's amplitudes for the overlaps, loaded before the last exchange so that their latency
    // overlaps it (slot 0 is final before a launch of the other slots; these loads precede this
    // block's own stores).
    // The tile is stored in the pass's store layout: the last round's when the planner chose
    // it (no exchange back), else the load layout.
    const int st_ri = pd->store_round;
    uint64_t gst = gthr;
    if (st_ri != pd->load_round) {
        uint32_t x = tid, m = prog.rounds[st_ri].reg_mask;
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const uint32_t b = (uint32_t)__builtin_ctz(m);
            const uint32_t lo = x & ((1u << b) - 1u);
            x = ((x ^ lo) << 1) | lo;
            m &= m - 1u;
        }
        gst = outer;
        for (int j = 0; j < K; ++j)
            if ((x >> j) & 1u) gst |= 1ull << pd->q_pos[j];
    }
    tv<R> refv[NR];
    const bool pre_ref = ovl != nullptr && slot != 0;
    if (pre_ref) {
#pragma unroll
        for (int r = 0; r < NR; ++r)
            refv[r] = *reinterpret_cast<const tv<R> *>(psi + 2 * (gst | pd->store_off[r]));
    }
    if (cur != prog.rounds[st_ri].reg_mask) exchange_to(prog.rounds[st_ri].reg_mask, st_ri);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        uint64_t i = gst | pd->store_off[r];
        if constexpr (sizeof(R) == 4) {
            typedef float f2 __attribute__((ext_vector_type(2)));
            __builtin_nontemporal_store(a[r], reinterpret_cast<f2 *>(base + 2 * i));
        } else {
            typedef double d2 __attribute__((ext_vector_type(2)));
            __builtin_nontemporal_store(a[r], reinterpret_cast<d2 *>(base + 2 * i));
        }
    }
    if (ovl) {
        // This tile's share of <psi_0|psi_slot> and <psi_slot|psi_slot> in FP64: the same sums
        // as the separate overlap reduction, one partial per (slot, tile).
        // Each product is one multiply-add into the running sum (for complex<float> the products
        // are exact in FP64, so this rounds once per term); the choice of reference is uniform,
        // so it is a branch rather than a select per amplitude.
        double v[3] = {0.0, 0.0, 0.0};
        if (pre_ref) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const double ar = refv[r].x, ai = refv[r].y, br = a[r].x, bi = a[r].y;
                v[0] = __builtin_fma(ai, bi, __builtin_fma(ar, br, v[0]));
                v[1] = __builtin_fma(-ai, br, __builtin_fma(ar, bi, v[1]));
                v[2] = __builtin_fma(bi, bi, __builtin_fma(br, br, v[2]));
            }
        } else {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const double br = a[r].x, bi = a[r].y;
                v[2] = __builtin_fma(bi, bi, __builtin_fma(br, br, v[2]));
            }
            v[0] = v[2];
        }
        // Block sums.  With more than one wave, every thread leaves its three sums in the LDS
        // (the tile's LDS, free once every wave has left the last exchange, holds three doubles
        // per thread when a thread keeps at least 16 bytes of amplitudes) and the first wave adds
        // them up, so the other waves finish without any cross-lane work.  A block of at most
        // one wave (or with too little LDS per thread) sums over its lanes, then over waves.
        constexpr bool kLdsSums = (sizeof(R) << (RB + 1)) >= 3 * sizeof(double);
        if (kLdsSums && nthr > 64u) {
            __syncthreads();
            double *sh = reinterpret_cast<double *>(smem);
#pragma unroll
            for (int k = 0; k < 3; ++k) sh[k * nthr + tid] = v[k];
            __syncthreads();
            if (tid < 64u) {
                double t[3] = {0.0, 0.0, 0.0};
                for (uint32_t j = tid; j < nthr; j += 64u)
#pragma unroll
                    for (int k = 0; k < 3; ++k) t[k] += sh[k * nthr + j];
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    for (int off = 32; off > 0; off >>= 1) t[k] += __shfl_xor(t[k], off, 64);
                if (tid == 0)
                    for (int k = 0; k < 3; ++k) ovl[bidx * 3 + k] = t[k];
            }
        } else {
            // wave sums (a block of fewer than 64 threads is one partial wave: sum over its lanes)
            const int width = nthr < 64u ? (int)nthr : 64;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                for (int off = width >> 1; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, width);
            if (nthr <= 64u) {
                if (tid == 0)
                    for (int k = 0; k < 3; ++k) ovl[bidx * 3 + k] = v[k];
            } else {
                __syncthreads();
                double *sh = reinterpret_cast<double *>(smem);
                if ((tid & 63u) == 0)
                    for (int k = 0; k < 3; ++k) sh[(tid >> 6) * 3 + k] = v[k];
                __syncthreads();
                if (tid < 3) {
                    double t = 0.0;
                    for (uint32_t w = 0; w < (nthr >> 6); ++w) t += sh[w * 3 + tid];
                    ovl[bidx * 3 + tid] = t;
                }
            }
        }
    }
}

// thread-safe one-time opt-in to the full 160 KiB of LDS
template <typename R, int RB, bool UNI, bool BLK, int ZV, bool MIX>
static hipError_t fused_attr_one()
{
    static const hipError_t attr = [] {
        // the kernel addresses its tile at LDS address 0: it must have no static LDS
        hipFuncAttributes fa;
        hipError_t e = hipFuncGetAttributes(&fa, (const void *)k_fused<R, RB, UNI, BLK, ZV, MIX>);
        if (e != hipSuccess) return e;
        if (fa.sharedSizeBytes != 0) return hipErrorInvalidKernelFile;
        return hipFuncSetAttribute((const void *)k_fused<R, RB, UNI, BLK, ZV, MIX>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    }();
    return attr;
}

template <typename R, int RB, bool UNI, int ZV>
static hipError_t fused_attr_mix()
{
    hipError_t e = fused_attr_one<R, RB, UNI, false, ZV, false>();
    if (e == hipSuccess) e = fused_attr_one<R, RB, UNI, false, ZV, true>();
    return e;
}

// the block-round variants (matrix-core rounds) exist for complex<float> with 16 registers only
template <typename R, int RB>
constexpr bool kBlockVariant = sizeof(R) == 4 && RB == 4;

template <typename R, int RB>
static hipError_t fused_attr()
{
    hipError_t e = fused_attr_mix<R, RB, false, 0>();
    if (e == hipSuccess) e = fused_attr_mix<R, RB, true, 0>();
    if (e == hipSuccess) e = fused_attr_mix<R, RB, false, 1>();
    if (e == hipSuccess) e = fused_attr_mix<R, RB, true, 1>();
    if (e == hipSuccess) e = fused_attr_mix<R, RB, false, 2>();
    if (e == hipSuccess) e = fused_attr_mix<R, RB, true, 2>();
    if (e == hipSuccess) e = fused_attr_one<R, RB, true, false, 3, false>();
    if (e == hipSuccess) e = fused_attr_mix<R, RB, false, 4>();
    if (e == hipSuccess) e = fused_attr_mix<R, RB, false, 6>();
    if (e == hipSuccess) e = fused_attr_one<R, RB, false, false, 5, true>();
    if constexpr (kBlockVariant<R, RB>) {
        // block rounds replace the op-by-op loop: no zero-input paths there
        if (e == hipSuccess) e = fused_attr_one<R, RB, false, true, 0, true>();
        if (e == hipSuccess) e = fused_attr_one<R, RB, true, true, 0, true>();
    }
    return e;
}

template <typename R, int RB, bool DEF = false>
static hipError_t launch_t(R *psi, int n, int S, const PassDesc &h, int pass_index, int rec_cap,
                           int64_t init, int64_t basis, const RunParams *dyn, ProgramDev prog, const void *rec,
                           const void *wtab, const uint64_t *otab, size_t lds, hipStream_t st,
                           double *ovl, int slot_base, int slots)
{
    const hipError_t attr = DEF ? hipSuccess : fused_attr<R, RB>();
    if (attr != hipSuccess) return attr;
    // the first pass may store every tile; otherwise a pass runs over the tiles that hold amplitude
    const bool fill = init >= 0 && h.zero_fill;
    const int free_bits = n - h.K - (fill ? 0 : __builtin_popcountll(h.classical));
    unsigned blocks = (unsigned)((uint64_t)(ovl ? slots : S) << free_bits);
    unsigned threads = 1u << (h.K - RB);
    uint32_t blocal = 0;
    for (int j = 0; j < h.K; ++j)
        if (((uint64_t)basis >> h.q_pos[j]) & 1ull) blocal |= 1u << j;
#define QS_FUSED_LAUNCH_M(UNI, BLK, ZV, MIX)                                                                   \
    hipLaunchKernelGGL((k_fused<R, RB, UNI, BLK, ZV, MIX>), dim3(blocks), dim3(threads), lds, st, psi, n, S, pass_index, \
                       rec_cap, init, basis, blocal, dyn, prog.passes, prog.stages, prog.rounds, prog.ops,         \
                       (const cxf<R> *)rec, (const cxf<R> *)wtab, otab, ovl, slot_base, slots)
    if constexpr (DEF) {
        const hipError_t e = fused_attr_one<R, RB, false, false, 7, true>();
        if (e != hipSuccess) return e;
        QS_FUSED_LAUNCH_M(false, false, 7, true);
        return hipGetLastError();
    } else {
#define QS_FUSED_LAUNCH(UNI, ZV)                                                                               \
    do {                                                                                                       \
        if (h.mixed_ops) QS_FUSED_LAUNCH_M(UNI, false, ZV, true);                                              \
        else QS_FUSED_LAUNCH_M(UNI, false, ZV, false);                                                         \
    } while (0)
    if constexpr (kBlockVariant<R, RB>) {
        if (h.blocks) {
            // block rounds: one variant, every op path kept
            if (h.uni_kernel) QS_FUSED_LAUNCH_M(true, true, 0, true);
            else QS_FUSED_LAUNCH_M(false, true, 0, true);
            return hipGetLastError();
        }
    }
    if (h.blocks) return hipErrorInvalidValue;   // no block-round variant for this tile shape
    if (h.zin_ops == 3) {
        QS_FUSED_LAUNCH_M(true, false, 3, false);
    } else if (h.zin_ops == 4) {
        if (h.shear) QS_FUSED_LAUNCH(false, 6);
        else QS_FUSED_LAUNCH(false, 4);
    } else if (h.zin_ops == 5) {
        QS_FUSED_LAUNCH_M(false, false, 5, true);
    } else if (h.zin_ops == 2) {
        if (h.uni_kernel) QS_FUSED_LAUNCH(true, 2);
        else QS_FUSED_LAUNCH(false, 2);
    } else if (h.zin_ops == 1) {
        if (h.uni_kernel) QS_FUSED_LAUNCH(true, 1);
        else QS_FUSED_LAUNCH(false, 1);
    } else {
        if (h.uni_kernel) QS_FUSED_LAUNCH(true, 0);
        else QS_FUSED_LAUNCH(false, 0);
    }
#undef QS_FUSED_LAUNCH
#undef QS_FUSED_LAUNCH_M
    return hipGetLastError();
    }
}

// One amplitude type's fused passes (fused_c64.hip, fused_c128.hip).
template <typename R>
hipError_t fused_attributes()
{
    hipError_t e;
    if ((e = fused_attr<R, 1>()) != hipSuccess || (e = fused_attr<R, 2>()) != hipSuccess ||
        (e = fused_attr<R, 3>()) != hipSuccess)
        return e;
    if ((e = fused_attr<R, 4>()) != hipSuccess || (e = fused_attr_one<R, 3, false, false, 7, true>()) != hipSuccess)
        return e;
    return fused_attr_one<R, 4, false, false, 7, true>();
}

template <typename R>
hipError_t fused_launch(R *p, int n, int S, const PassDesc &h, int pass_index, int rec_cap, int64_t init, int64_t basis,
                        const RunParams *dyn, ProgramDev prog, const void *rec, const void *wtab, const uint64_t *otab,
                        size_t lds, hipStream_t st, double *ovl, int slot_base, int slots)
{
#define QS_FUSED_CASE(RB)                                                                                            \
    case RB:                                                                                                        \
        return launch_t<R, RB>(p, n, S, h, pass_index, rec_cap, init, basis, dyn, prog, rec, wtab, otab, lds, st, ovl, \
                               slot_base, slots);
    // (The collecting variants last, so that their kernels are compiled, and placed, after the others: ahead
    // of the 16-register kernels, whose code is larger than the instruction cache, the 8-register one cost
    // brickwork passes at n = 26, complex<double>, 0.7 %.)
    switch (h.defer ? h.RB + 8 : h.RB) {
        QS_FUSED_CASE(1)
        QS_FUSED_CASE(2)
        QS_FUSED_CASE(3)
        QS_FUSED_CASE(4)
    case 11:
        return launch_t<R, 3, true>(p, n, S, h, pass_index, rec_cap, init, basis, dyn, prog, rec, wtab, otab, lds, st,
                                    ovl, slot_base, slots);
    case 12:
        return launch_t<R, 4, true>(p, n, S, h, pass_index, rec_cap, init, basis, dyn, prog, rec, wtab, otab, lds, st,
                                    ovl, slot_base, slots);
    }
#undef QS_FUSED_CASE
    return hipErrorInvalidValue;
}

}  // namespace qs
