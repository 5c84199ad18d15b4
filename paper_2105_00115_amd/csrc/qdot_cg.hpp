// Device side of conjugate gradient (Alg. 4) run by a gang of blocks inside
// one launch; used by the single-system CG launch and by the batched launch.
//
// A gang of G blocks of NT threads solves one system; block b of the gang
// owns a contiguous slice of rows and every vector update, SpMV row and qdot
// pass on that slice.  Gang barriers separate the steps that need data from
// other slices:
//   before the SpMV (p complete), after a qdot's pass 1 (histogram merged),
// three per iteration (one more for an inner product that the guaranteed
// mode sums again), and block 0 gathers and publishes each qdot's value.
//
// An iteration is a chain of latencies: each barrier costs several round
// trips to the memory that all XCDs share (0.7 to 1 us each), so they are kept
// few.  The counters of a barrier only ever count up (no resets, and a block
// knows the generation it waits for without reading it); blocks arrive in
// groups, and poll their group's own copy of the release word.  The
// histograms of a group are added to the gang's by the group's last block
// while the other groups still arrive; every block then reads the merged
// counts in one round trip, whole, and selects the classes itself.  After the
// sweep there is no barrier: block 0 polls the blocks' partials themselves and
// combines them as they come in, and the word that the others poll is the
// inner product.
// Poisson 1024^2, per iteration with the two-pass qdot: 87 us with counters
// reset at each barrier, a whole-gang merge and combine by the last block and
// 512 blocks of 256 threads; 64 us with the barriers above; 53.7 us with the
// matrix's resident rows, 51.4 with block 0 polling the sums, 50.1 with each
// thread's next row ahead (all below).  With the FP64 dot: 48 -> 32.8 us.
// Every block holds bit-identical scalars (alpha, beta, c) and takes the same
// branches: no decision is broadcast.  Two buffers alternate between
// consecutive qdots.
//
// Every wait is bounded: a barrier that does not complete within the spin
// limit raises the gang's abort flag, every block leaves, and the call
// reports QDOT_E_DEVICE.  A block leaves its LDS as the next item of its
// launch expects it.  The launches size their grids so that all blocks
// of a gang are resident together.
#pragma once
#include <cmath>

#include "qdot_select.hpp"

namespace qd {

struct CgSys {
    int64_t n;
    const int32_t *rowptr;
    const int32_t *col;
    const double *val;
    const double *b;
    double *x;
    double *r, *p, *q;  // scratch, n each
    double rtol, qtol;
    int maxit, use_qdot;
    qdot_result *trace;  // nullable: 2 * maxit + 1 results
};

constexpr int MAX_GANG = 512;
constexpr int BAR_GROUPS = 8;     // groups of a large gang: block gb in group gb mod 8
constexpr int BAR_ONE_LEVEL = 64; // gangs up to this size are one group

struct GangLine {  // a word, or two, on a 128-byte line of their own
    unsigned int v;
    unsigned int pad;
    unsigned long long w;
    unsigned int fill[28];
};

struct GangQ {  // per gang and qdot buffer; zero between its uses
    // a large gang's groups: the counts of one group's blocks each
    uint4 hist[BAR_GROUPS][FQ];
    // the gang's counts (slots, and the four counts behind them)
    uint4 hm[FQ];
};

// The word in place of a value that is not there yet: a NaN that no sum has.
constexpr unsigned long long NO_VALUE = 0x7ff4dead00c0ffeeull;

struct Gang {
    unsigned int abort;
    unsigned int spin_limit;
    unsigned int join_spins;      // polls of gang_join
    unsigned int pad[29];
    GangLine join;                // .v: blocks that are on the chip (gang_join)
    GangLine verdict;             // .v: what became of that
    GangLine sub[BAR_GROUPS];     // .v: arrivals of a group's blocks
    GangLine top;                 // .v: arrivals of the groups
    GangLine gen[BAR_GROUPS];     // .v: the group's copy of the generation
    GangLine val[2][BAR_GROUPS];  // .w: the group's copy of dot buffer k's value
    GangQ qb[2];
    double partials[2][MAX_GANG * 6];  // NO_VALUE between their uses
    // partials[k] combined in block order by block 0
    double pfin[2][6];
    // one-pass mode: per block the live slot range, zero count and non-finite
    // flag, and the result of buffer k's qdot, published by the last block to
    // arrive
    int4 rec[2][MAX_GANG];
    qdot_result res[2];
};

// A gang that has a launch of its own first waits until all of its blocks are
// on the chip: another launch of this kind (a solve on another stream) may
// have taken some CUs in between, and each would then wait for the CUs that
// the other holds.  A gang that has not come together after join_spins polls
// leaves the chip again, before it has touched anything, and the host launches
// it anew: JOIN_SPINS of them (some 20 ms) at first, and twice as many each
// time, so that long blocks of other work, which a gang has to wait out, hold
// it up no longer than if it had stayed.  `status` gets NOT_RESIDENT then.  The
// verdict is given once: by the last block to join, or by the first to give up.
// 0.2 % of a solve of 60 iterations.
constexpr unsigned int JOIN_SPINS = 1u << 14;
constexpr unsigned int JOIN_GO = 1u, JOIN_LEAVE = 2u;
constexpr int32_t NOT_RESIDENT = 0x7e51;  // none of the statuses that a caller sees

__device__ __forceinline__ bool gang_join(Gang *gg, int G, int32_t *status)
{
    __shared__ int s_go;
    if (threadIdx.x == 0) {
        unsigned int v = 0u;
        auto give = [&](unsigned int mine) {
            v = 0u;
            if (__hip_atomic_compare_exchange_strong(&gg->verdict.v, &v, mine, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                v = mine;
                if (mine == JOIN_LEAVE) st_dev(status, NOT_RESIDENT);
            }
        };
        if (__hip_atomic_fetch_add(&gg->join.v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
                1u == (unsigned)G) {
            give(JOIN_GO);
        } else {
            const unsigned int limit = gg->join_spins;
            for (unsigned int spins = 0; (v = ld_dev(&gg->verdict.v)) == 0u; spins++) {
                if (spins >= limit) {
                    give(JOIN_LEAVE);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        s_go = v == JOIN_GO;
    }
    __syncthreads();
    return s_go != 0;
}

// A block's view of its gang.  gen: barriers passed since the gang was reset.
struct GangCtx {
    Gang *gg;
    int G, gb, groups, grp;
    unsigned int members;  // blocks of the group
    unsigned int gen;
};

__device__ __forceinline__ GangCtx gang_enter(Gang *gg, int G, int gb)
{
    GangCtx c;
    c.gg = gg;
    c.G = G;
    c.gb = gb;
    c.groups = G > BAR_ONE_LEVEL ? BAR_GROUPS : 1;
    c.grp = gb % c.groups;
    c.members = (unsigned)((G - c.grp + c.groups - 1) / c.groups);
    // no block of the gang can pass a barrier before all have read it
    c.gen = ld_dev(&gg->gen[c.grp].v);
    return c;
}

// ---------------------------------------------------------------------------
// Gang barrier.  Everything a block hands to the others (vector entries,
// histogram merges, partials, clears) is written with device-scope atomics
// or write-through stores and read with device-scope loads, so arriving
// needs only the block's own memory operations to have completed
// (vmem_drain) and leaving needs no cache invalidation.  The barrier numbered
// gen is complete when each group's counter has reached (gen + 1) * members
// and the groups' counter (gen + 1) * groups.
//
// group_work() is run by the last block of a large gang's group before the
// group counts as arrived.  Returns true in every thread of the last block to
// arrive; what that block has done by then, and does before it releases the
// others, happens once for the gang.
template <bool GW, class GroupWork>
__device__ __forceinline__ bool gang_arrive(const GangCtx &c, GroupWork &&group_work)
{
    __shared__ int s_last;
    vmem_drain();
    __syncthreads();
    Gang *gg = c.gg;
    auto count = [](unsigned int *w) {
        return __hip_atomic_fetch_add(w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
    };
    if (threadIdx.x == 0) {
        bool last = count(&gg->sub[c.grp].v) == (c.gen + 1u) * c.members;
        if (!GW && last && c.groups > 1)
            last = count(&gg->top.v) == (c.gen + 1u) * (unsigned)c.groups;
        s_last = last;
    }
    __syncthreads();
    bool last = s_last != 0;
    if (GW && last && c.groups > 1) {
        group_work();
        vmem_drain();
        __syncthreads();
        if (threadIdx.x == 0) s_last = count(&gg->top.v) == (c.gen + 1u) * (unsigned)c.groups;
        __syncthreads();
        last = s_last != 0;
    }
    return last;
}

// Polls until ready() or the spin limit; false when the gang has given up.
template <class Ready>
__device__ __forceinline__ bool gang_poll(Gang *gg, Ready &&ready)
{
    unsigned int spins = 0;
    while (!ready()) {
        if ((++spins & 63u) == 0u && (ld_dev(&gg->abort) || spins > gg->spin_limit)) {
            __hip_atomic_fetch_or(&gg->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return true;
}

// The barrier; the last block to arrive runs work() with all its threads
// before it releases the others.
template <bool GW, class GroupWork, class Work>
__device__ __forceinline__ bool gang_barrier_with(GangCtx &c, GroupWork &&group_work, Work &&work)
{
    __shared__ int s_ok;
    Gang *gg = c.gg;
    const unsigned int next = c.gen + 1u;
    if (gang_arrive<GW>(c, group_work)) {
        work();
        vmem_drain();
        __syncthreads();
        if ((int)threadIdx.x < c.groups) st_dev(&gg->gen[threadIdx.x].v, next);
        c.gen = next;
        return true;
    }
    if (threadIdx.x == 0) s_ok = gang_poll(gg, [&] { return ld_dev(&gg->gen[c.grp].v) == next; });
    __syncthreads();
    c.gen = next;
    return s_ok != 0;
}

template <class Work>
__device__ __forceinline__ bool gang_barrier_then(GangCtx &c, Work &&work)
{
    return gang_barrier_with<false>(c, [] {}, work);
}

__device__ __forceinline__ bool gang_barrier(GangCtx &c)
{
    return gang_barrier_then(c, [] {});
}

// Hands out one value to the gang (buffer k): in block 0, work(ok) returns it
// in thread 0; the others poll for it.  Block 0 publishes once every block has
// contributed to the value, so every block is past its use of the other
// buffer's value: block 0 has to have taken that back (gang_retract, with a
// drain after it) before it publishes.
template <class Work>
__device__ __forceinline__ bool gang_publish(const GangCtx &c, int k, double &value, Work &&work)
{
    __shared__ int s_ok;
    __shared__ double s_v;
    Gang *gg = c.gg;
    if (c.gb == 0) {
        bool ok = true;
        const double v = work(ok);
        if (threadIdx.x == 0) {
            s_v = v;
            s_ok = ok;
        }
        __syncthreads();
        unsigned long long bits = (unsigned long long)__double_as_longlong(s_v);
        if (bits == NO_VALUE) bits = 0x7ff8000000000000ull;
        if ((int)threadIdx.x < c.groups && s_ok) st_dev(&gg->val[k][threadIdx.x].w, bits);
    } else if (threadIdx.x == 0) {
        unsigned long long bits = NO_VALUE;
        s_ok = gang_poll(gg, [&] {
            bits = ld_dev(&gg->val[k][c.grp].w);
            return bits != NO_VALUE;
        });
        s_v = __longlong_as_double((long long)bits);
    }
    __syncthreads();
    value = s_v;
    const bool ok = s_ok != 0;
    __syncthreads();
    return ok;
}

// Block 0 takes back the value of the buffer other than k.
__device__ __forceinline__ void gang_retract(const GangCtx &c, int k)
{
    if ((int)threadIdx.x < c.groups) st_dev(&c.gg->val[k ^ 1][threadIdx.x].w, NO_VALUE);
}

// The words w of a block's partials as soon as it has stored them (they hold
// NO_VALUE before), taken back at once: the words are their own flags, so a
// block stores them and needs no drain and no counter.  valid: the calling
// thread has words to wait for.
template <int NW>
__device__ __forceinline__ bool gang_take(const GangCtx &c, unsigned long long *const (&w)[NW],
                                          bool valid, double (&out)[NW])
{
    unsigned long long bits[NW];
    bool ok = true;
    if (valid) {
        ok = gang_poll(c.gg, [&] {
            bool all = true;
#pragma unroll
            for (int i = 0; i < NW; i++) {
                bits[i] = ld_dev(w[i]);
                all &= bits[i] != NO_VALUE;
            }
            return all;
        });
#pragma unroll
        for (int i = 0; i < NW; i++) {
            out[i] = __longlong_as_double((long long)bits[i]);
            st_dev(w[i], NO_VALUE);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NW; i++) out[i] = 0.0;
    }
    return ok;
}

struct DotOut {
    double value;
    bool all_perf;  // qdot perforated every component of a nonzero vector
    bool ok;        // gang still healthy
};

// Shared-memory workspace of one block (CG and batched kernels).
template <int NT>
struct CgLdsT {
    // the key slots and the counts behind them (qdot_select.hpp); zero
    // between the uses
    alignas(16) unsigned int h[4 * FQ];
    unsigned char lut[W_LUT];
    Acc red[3][NT / 64];
    int4 scratch[NT / 64];
    SelLds<NT> sel;
    qdot_result res;
};

// Pass 1 of qdot for one component pair, into the block's LDS histogram h.
__device__ __forceinline__ void scan_pair(double a, double b, int key_mode, unsigned int *h,
                                          unsigned int &sg)
{
    const Comp c = component(a, b, key_mode);
    sg |= c.zero ? 0u : (c.sgn ? 1u : 2u);
    atomicAdd(&h[c.slot + (c.bad ? 1 : 0)], 1u);
}

// Groups of 4 NT components in flight per thread in a gang's sweeps: a large
// block's slice is one group.
template <int NT>
constexpr int gang_u()
{
    return NT >= 1024 ? 1 : 2;
}

// The waves' sums of the three classes (red, per wave) merged in the first
// wave: lane 16 q holds class q's.  A barrier precedes it.
template <int NT>
__device__ __forceinline__ Acc merge_waves(Acc (*red)[NT / 64])
{
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, q = lane >> 4, w = lane & 15;
    Acc a = {0.0, 0.0};
    if (q < 3 && w < NW) a = red[q][w];
    if (NW > 8) a = acc_dpp<DPP_FROM8>(a);
    if (NW > 4) a = acc_dpp<DPP_FROM4>(a);
    a = acc_dpp<DPP_FROM2>(a);
    return acc_dpp<DPP_FROM1>(a);
}

// a.b over the gang's rows by qdot (buffer k), value identical in every block.
// With `scanned` the caller has already put its rows' keys into L.h (while
// it produced a or b) and passes its sign bits.  L.h is zero again afterwards.
// trace_slot: where this block writes the whole result, or NULL; with_trace:
// some block of the gang does.
//
// GUARD (guard_mode 1): after the combine every block evaluates the lower
// bound of Thm 3.4 from its copy of the counts and its class table, and
// certifies the result or reselects against E_lo (or makes every bin
// double) and sums its rows again, into the other partials buffer (free:
// every block has read it in the previous inner product), then checks again
// with the larger lower bound: the steps and flags of the single-vector
// guaranteed mode, one more gang barrier when it reselects.
template <bool GUARD, int NT>
__device__ __forceinline__ DotOut gang_qdot(const double *a, const double *bv, int64_t n,
                                            int64_t r0, int64_t r1, const SelArgs &sa,
                                            GangCtx &c, int k, CgLdsT<NT> &L,
                                            qdot_result *trace_slot, bool with_trace,
                                            bool scanned = false, unsigned int sg = 0)
{
    constexpr int U = gang_u<NT>();
    constexpr int K = (FQ + NT - 1) / NT;
    DotOut o = {0.0, false, true};
    Gang *gg = c.gg;
    GangQ &Q = gg->qb[k];
    const int tid = threadIdx.x;
    uint4 *h4 = reinterpret_cast<uint4 *>(L.h);
    const bool vec = ((((uintptr_t)a) | ((uintptr_t)bv)) & 15) == 0;
    auto sweep_rows = [&](auto &&body) {
        if (vec) stream_strided<true, U, NT>(a, bv, r0, (int64_t)U * NT * EPT, r1, body);
        else stream_strided<false, U, NT>(a, bv, r0, (int64_t)U * NT * EPT, r1, body);
    };
    if (!scanned)
        sweep_rows([&](const double *xv, const double *yv, int64_t, int lim) {
            count4(xv, yv, lim, sa.key_mode, L.h, sg);
        });
    count_signs(sg, L.h);
    select_begin(L.sel);
    __syncthreads();
    // the block's counts into its group's, or a small gang's own
    {
        unsigned int *gh =
            reinterpret_cast<unsigned int *>(c.groups > 1 ? Q.hist[c.grp] : Q.hm);
        for (int j = tid; j < 4 * FQ; j += NT) {
            const unsigned int v = L.h[j];
            if (v)
                __hip_atomic_fetch_add(&gh[j], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // a group's last block adds the group's counts to the gang's and clears
    // them for the qdot after next
    auto merge_group = [&]() {
        unsigned int *gh = reinterpret_cast<unsigned int *>(Q.hist[c.grp]);
        unsigned int *gm = reinterpret_cast<unsigned int *>(Q.hm);
        unsigned int m[4 * K];
#pragma unroll
        for (int i = 0; i < 4 * K; i++) {
            const int j = i * NT + tid;
            m[i] = j < 4 * FQ ? ld_dev(&gh[j]) : 0u;
        }
#pragma unroll
        for (int i = 0; i < 4 * K; i++) {
            const int j = i * NT + tid;
            if (m[i]) {
                __hip_atomic_fetch_add(&gm[j], m[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                st_dev(&gh[j], 0u);
            }
        }
    };
    if (!gang_barrier_with<true>(c, merge_group, [] {})) {
        o.ok = false;
        return o;
    }
    // the merged counts into LDS, and the selection, in every block
    {
        uint4 v[K];
#pragma unroll
        for (int i = 0; i < K; i++) {
            const int q = i * NT + tid;
            v[i] = q < FQ ? ld_dev_quad(&Q.hm[q]) : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int i = 0; i < K; i++)
            if (i * NT + tid < FQ) h4[i * NT + tid] = v[i];
        find_window<NT, K>(v, L.sel);
    }
    __syncthreads();
    const Sel s = select_classes<NT>(L.h, sa, L.sel, L.lut);
    const int lo = s.n_bins ? s.e_min - KMIN : W, hi = s.n_bins ? s.e_max - KMIN : -1;
    auto clear_counts = [&]() {
        unsigned int *gm = reinterpret_cast<unsigned int *>(Q.hm);
        for (int j = lo + tid; j <= hi; j += NT) st_dev(&gm[j], 0u);
        if (tid < 4) st_dev(&gm[W + tid], 0u);
    };
    // pass 2 over own rows into partials buffer kp
    auto sweep = [&](int e_max, int c32, int kp) {
        Acc acc[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
        sweep_rows([&](const double *xv, const double *yv, int64_t, int lim) {
            acc_group<false>(xv, yv, lim, L.lut, sa.key_mode, e_max, c32, true, acc[0], acc[1],
                             acc[2], nullptr);
        });
        block_reduce3_waves<NT, false>(acc, L.red);
        __syncthreads();
        if (tid < 64) {
            const Acc b = merge_waves<NT>(L.red);
            const int q = tid >> 4;
            if ((tid & 15) == 0 && q < 3) {
                double *pp = gg->partials[kp];
                st_dev(&pp[(2 * q) * c.G + c.gb], b.s);
                st_dev(&pp[(2 * q + 1) * c.G + c.gb], b.c);
            }
        }
    };
    // block 0: the gang's partials in block order, as they come in; the
    // classes' sums into pfin when someone will read them, and the combined
    // value in thread 0
    __shared__ int s_lost;
    auto combine = [&](int e_max, int c32, int kp, bool &ok) -> double {
        if (tid == 0) s_lost = 0;
        __syncthreads();
        Acc f[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
        unsigned long long *pp = reinterpret_cast<unsigned long long *>(gg->partials[kp]);
        for (int b0 = 0; b0 < c.G; b0 += NT) {
            const int b = b0 + tid;
            unsigned long long *const w[6] = {&pp[b],           &pp[c.G + b],     &pp[2 * c.G + b],
                                              &pp[3 * c.G + b], &pp[4 * c.G + b], &pp[5 * c.G + b]};
            double d[6];
            if (!gang_take(c, w, b < c.G, d)) s_lost = 1;
#pragma unroll
            for (int q = 0; q < 3; q++) f[q] = acc_merge(f[q], Acc{d[2 * q], d[2 * q + 1]});
        }
        block_reduce3_waves<NT, true>(f, L.red);
        __syncthreads();
        ok = !s_lost;
        double v = 0.0;
        if (tid < 64) {
            const Acc b = merge_waves<NT>(L.red);
            Acc t[3];
#pragma unroll
            for (int q = 0; q < 3; q++) t[q] = lane_acc(b, 16 * q);
            if (tid == 0) {
                if (GUARD || with_trace) {
                    for (int q = 0; q < 3; q++) {
                        st_dev(&gg->pfin[kp][2 * q], t[q].s);
                        st_dev(&gg->pfin[kp][2 * q + 1], t[q].c);
                    }
                    vmem_drain();
                }
                combine_value(t, e_max, c32, 0, &L.sel.sums);
                v = L.sel.sums.value;
            }
        }
        return v;
    };
    // the whole result in this block's L.res, for the guard and the trace
    auto fill_result = [&]() {
        select_count<NT>(L.h, s, sa, L.sel);
        __syncthreads();
        if (tid == 0) {
            result_fields<NT>(s, sa, n, L.sel, L.res);
            L.sel.sum = 0.0;
            if (s.live() && s.kept) {
                Acc f[3];
                for (int q = 0; q < 3; q++)
                    f[q] = Acc{ld_dev(&gg->pfin[k][2 * q]), ld_dev(&gg->pfin[k][2 * q + 1])};
                L.sel.sum = combine_value(f, s.e_max, s.c32, L.res.flags, &L.res);
            }
        }
        __syncthreads();
    };
    const bool swept = s.live() && s.kept;
    if (swept) {
        // every block has passed the barrier, and so the other value
        if (c.gb == 0) gang_retract(c, k);
        sweep(s.e_max, s.c32, k);
        if (c.gb == 0) vmem_drain();
        if (!gang_publish(c, k, o.value,
                          [&](bool &ok) { return combine(s.e_max, s.c32, k, ok); })) {
            o.ok = false;
            return o;
        }
        // every block has read the merged counts; they are zero again before
        // block 0 arrives at its next barrier
        if (c.gb == 0) clear_counts();
    } else {
        // nothing to sum: every block knows the value
        o.value = s.status != QDOT_OK ? __longlong_as_double(0x7ff8000000000000ll) : 0.0;
        if (!gang_barrier_then(c, [&] {
                gang_retract(c, k);
                clear_counts();
            })) {
            o.ok = false;
            return o;
        }
    }
    bool all_perf = s.live() && !s.kept;
    if constexpr (GUARD) {
        __shared__ int s_go, s_dref, s_passes;
        __shared__ double s_low;
        fill_result();
        if (tid == 0) {
            s_go = L.res.status == QDOT_OK && L.res.n_bins > 0;
            // every product zero: +0 is exact
            if (L.res.status == QDOT_OK && L.res.n_bins == 0) L.res.flags |= QDOT_F_GUARANTEED;
            s_dref = 0;
            s_passes = L.res.passes;
        }
        __syncthreads();
        if (s_go) {
            const int e_max = L.res.e_max;
            auto get = [&](int j) { return (unsigned long long)L.h[j]; };
            auto put = [&](int j, int cls) { L.lut[j] = (unsigned char)cls; };
            auto noclear = [&](int) {};
            const GuardSums g0 = guard_sums<NT>(get, L.lut, lo, hi, e_max);
            if (tid == 0) {
                const double low = guard_lower(g0, L.sel.sum, n, s.signs);
                if (guard_certified(L.res.bound_rel, low, sa.tol)) {
                    L.res.flags |= QDOT_F_GUARANTEED;
                    L.res.lower = ldexp(low, e_max);
                } else {
                    // L <= 0: every bin double (scores >= 23, one more
                    // non-strict)
                    const int ref = low > 0.0 ? e_max + ilogb(low)
                                              : L.res.e_min - L.res.t - 22 - sa.nonstrict;
                    if (ref < e_max) {
                        s_dref = e_max - ref;
                        s_low = low;
                    } else {
                        L.res.lower = low > 0.0 ? ldexp(low, e_max) : 0.0;
                    }
                }
            }
            __syncthreads();
            if (s_dref) {
                // reselection against e_ref = e_max - dref, second sweep
                const CutParams p2 = block_cutoff<NT>(lo, hi, s.n_zero, 0u, n, sa.tol,
                                                      sa.score_mode, sa.nonstrict, get, put,
                                                      noclear, &L.res, nullptr, s_dref);
                if (tid == 0) {
                    L.res.flags |= QDOT_F_RESELECTED;
                    L.res.passes = s_passes + (p2.skip ? 0 : 1);
                    L.sel.sum = 0.0;
                }
                if (!p2.skip) {
                    sweep(p2.e_max, p2.c32, k ^ 1);
                    bool ok = true;
                    if (c.gb == 0) (void)combine(p2.e_max, p2.c32, k ^ 1, ok);
                    if (!gang_barrier(c) || !ok) {
                        o.ok = false;
                        return o;
                    }
                    if (tid == 0) {
                        Acc f[3];
                        for (int q = 0; q < 3; q++)
                            f[q] = Acc{ld_dev(&gg->pfin[k ^ 1][2 * q]),
                                       ld_dev(&gg->pfin[k ^ 1][2 * q + 1])};
                        L.sel.sum = combine_value(f, p2.e_max, p2.c32,
                                                  p2.flags | QDOT_F_RESELECTED, &L.res);
                    }
                }
                __syncthreads();
                const GuardSums g1 = guard_sums<NT>(get, L.lut, lo, hi, e_max);
                if (tid == 0) {
                    const double low = fmax(guard_lower(g1, L.sel.sum, n, s.signs), s_low);
                    L.res.flags |= QDOT_F_RESELECTED |
                                   (guard_certified(L.res.bound_rel, low, sa.tol)
                                        ? QDOT_F_GUARANTEED
                                        : 0);
                    L.res.lower = low > 0.0 ? ldexp(low, e_max) : 0.0;
                }
            }
        }
        __syncthreads();
        o.value = L.res.value;
        all_perf = (L.res.flags & QDOT_F_ALL_PERF) && L.res.n_bins > 0;
    } else if (trace_slot) {
        fill_result();
    }
    o.all_perf = all_perf;
    if (tid == 0 && trace_slot) *trace_slot = L.res;
    // the LDS counts back to zero for the next scan (all of them: with zero
    // or non-finite products alone there is no live window)
    __syncthreads();
    for (int j = lo + tid; j <= hi; j += NT) L.h[j] = 0u;
    if (tid < 4) L.h[W + tid] = 0u;
    __syncthreads();
    return o;
}

// a.b over the gang's rows by the one-pass qdot (accum_mode 1, value as the
// exact sum of the kept leaves), buffer k, value identical in every block.
// Each block reads its rows once: keys into its LDS histogram and, for the
// bins within `depth` of its running maximum, the candidate sums of every
// precision into its LDS window (s1_stream), which it adds into the gang's
// table `tab` (W x S1_PIECES sums, exact in any order, zero between calls).
// The last block to arrive at the one barrier merges the records and the
// histogram copies, selects, picks each kept bin's sum from the table,
// clears the copies and the table over the live window and publishes the
// result; the others read it.  No class table or second sweep is needed
// outside that block, so an inner product costs one gang barrier.
__device__ __forceinline__ DotOut gang_qdot_s1(const double *a, const double *bv, int64_t n,
                                               int64_t r0, int64_t r1, double tol, int key_mode,
                                               int score_mode, int nonstrict, GangCtx &c, int k,
                                               CgLdsT<BLOCK> &L, S1Lds &S1, double *tab,
                                               qdot_result *trace_slot)
{
    DotOut o = {0.0, false, true};
    Gang *gg = c.gg;
    const int G = c.G, gb = c.gb;
    unsigned int *gh = reinterpret_cast<unsigned int *>(gg->qb[k].hist[gb % BAR_GROUPS]);
    const bool vec = ((((uintptr_t)a) | ((uintptr_t)bv)) & 15) == 0;
    // admitted by the host: depth <= S1_WIN
    const int depth = s1_depth_dev(n, tol, score_mode);
    unsigned int nz = 0, bad = 0;
    S1Run run = s1_run_start();
    s1_begin(S1);
    __syncthreads();
    if (r1 > r0) {
        if (vec)
            s1_stream<true, 2>(a + r0, bv + r0, 0, 2 * CHUNK, r1 - r0, key_mode, depth, L.h, S1,
                               run, nz, bad);
        else
            s1_stream<false, 2>(a + r0, bv + r0, 0, 2 * CHUNK, r1 - r0, key_mode, depth, L.h,
                                S1, run, nz, bad);
    }
    const int top = run.top;
    __syncthreads();
    int lo = W, hi = -1;
    for (int j = threadIdx.x; j < W; j += BLOCK) {
        const unsigned int v = L.h[j];
        if (v) {
            __hip_atomic_fetch_add(&gh[j], v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            L.h[j] = 0u;
            lo = min(lo, j);
            hi = max(hi, j);
        }
    }
    if (threadIdx.x == 0) L.h[W] = 0u;
    if (top >= 0)
        for (int i = threadIdx.x; i < depth * S1_PIECES; i += BLOCK) {
            const int bin = top - i / S1_PIECES;
            if (bin < 0) continue;
            const double v = S1.win[bin & (S1_WIN - 1)][i % S1_PIECES];
            if (v != 0.0)
                __hip_atomic_fetch_add(&tab[(size_t)bin * S1_PIECES + i % S1_PIECES], v,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    unsigned int bs = bad ? 1u : 0u;
    block_reduce_range(lo, hi, nz, bs, L.scratch);
    if (threadIdx.x == 0) {
        int *rec = &gg->rec[k][gb].x;
        st_dev(rec, lo);
        st_dev(rec + 1, hi);
        st_dev(rec + 2, (int)nz);
        st_dev(rec + 3, (int)bs);
    }
    auto finish = [&]() {
        gang_retract(c, k);
        int lo2 = W, hi2 = -1;
        unsigned int z2 = 0, bs2 = 0;
        for (int b = threadIdx.x; b < G; b += BLOCK) {
            const int *rec = &gg->rec[k][b].x;
            lo2 = min(lo2, ld_dev(rec));
            hi2 = max(hi2, ld_dev(rec + 1));
            z2 += (unsigned int)ld_dev(rec + 2);
            bs2 |= (unsigned int)ld_dev(rec + 3);
        }
        block_reduce_range(lo2, hi2, z2, bs2, L.scratch);
        const int ncopy = min(G, BAR_GROUPS);
        for (int j = lo2 + (int)threadIdx.x; j <= hi2; j += BLOCK) {
            unsigned int v = 0u;
            for (int q = 0; q < ncopy; q++) {
                unsigned int *hq = reinterpret_cast<unsigned int *>(gg->qb[k].hist[q]);
                v += ld_dev(&hq[j]);
                st_dev(&hq[j], 0u);
            }
            L.h[j] = v;
        }
        __syncthreads();
        auto get = [&](int j) { return (unsigned long long)L.h[j]; };
        auto put = [&](int j, int c) { L.lut[j] = (unsigned char)c; };
        auto noclear = [&](int) {};
        const CutParams p = block_cutoff<BLOCK>(lo2, hi2, z2, bs2 & 1u, n, tol, score_mode,
                                                nonstrict, get, put, noclear, &L.res, nullptr);
        if (!p.skip)
            s1_pick(p.e_max, max(lo2, p.e_max - KMIN - depth + 1), p.flags, L.lut,
                    [&](int bin, int q) { return ld_dev(&tab[(size_t)bin * S1_PIECES + q]); },
                    L.red, &L.res);
        __syncthreads();
        // the table and the LDS copy back to zero over the live window
        if (hi2 >= lo2) {
            for (int i = lo2 * S1_PIECES + (int)threadIdx.x; i < (hi2 + 1) * S1_PIECES;
                 i += BLOCK)
                st_dev(&tab[i], 0.0);
            for (int j = lo2 + (int)threadIdx.x; j <= hi2; j += BLOCK) L.h[j] = 0u;
        }
        constexpr int NWORD = (int)(sizeof(qdot_result) / sizeof(unsigned long long));
        if (threadIdx.x < NWORD)
            st_dev(reinterpret_cast<unsigned long long *>(&gg->res[k]) + threadIdx.x,
                   reinterpret_cast<const unsigned long long *>(&L.res)[threadIdx.x]);
    };
    if (!gang_barrier_then(c, finish)) {
        o.ok = false;
        return o;
    }
    constexpr int NWORD = (int)(sizeof(qdot_result) / sizeof(unsigned long long));
    if (threadIdx.x < NWORD)
        reinterpret_cast<unsigned long long *>(&L.res)[threadIdx.x] =
            ld_dev(reinterpret_cast<const unsigned long long *>(&gg->res[k]) + threadIdx.x);
    __syncthreads();
    o.value = L.res.value;
    o.all_perf = (L.res.flags & QDOT_F_ALL_PERF) && L.res.n_bins > 0;
    if (threadIdx.x == 0 && trace_slot) *trace_slot = L.res;
    __syncthreads();
    return o;
}

// a.b over the gang's rows in plain FP64 (buffer k): the blocks' sums added in
// a fixed order by the last block to arrive.
template <int NT>
__device__ __forceinline__ DotOut gang_dot64(const double *a, const double *bv, int64_t r0,
                                             int64_t r1, GangCtx &c, int k, CgLdsT<NT> &L)
{
    DotOut o = {0.0, false, true};
    Gang *gg = c.gg;
    const int tid = threadIdx.x;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t i = r0 + tid;
    for (; i + 3 * NT < r1; i += 4 * NT) {
#pragma unroll
        for (int u = 0; u < 4; u++) s[u] = fma(a[i + u * NT], bv[i + u * NT], s[u]);
    }
    for (; i < r1; i += NT) s[0] = fma(a[i], bv[i], s[0]);
    auto block_sum = [&](double v) {
        v = wave_sum_d(v);
        if ((tid & 63) == 0) L.red[0][tid >> 6].s = v;
        __syncthreads();
        double f = 0.0;
        if (tid == 0) {
            f = L.red[0][0].s;
            for (int w = 1; w < NT / 64; w++) f += L.red[0][w].s;
        }
        __syncthreads();
        return f;
    };
    const double part = block_sum((s[0] + s[1]) + (s[2] + s[3]));
    if (tid == 0) st_dev(&gg->partials[k][c.gb], part);
    o.ok = gang_publish(c, k, o.value, [&](bool &ok) {
        double v = 0.0;
        bool mine = true;
        for (int b0 = 0; b0 < c.G; b0 += NT) {
            unsigned long long *const w[1] = {
                reinterpret_cast<unsigned long long *>(&gg->partials[k][b0 + tid])};
            double d[1];
            mine &= gang_take(c, w, b0 + tid < c.G, d);
            v += d[0];
        }
        // a wave's own blocks having contributed says nothing about the others':
        // the other value goes once every wave has its blocks' sums
        ok = __syncthreads_and(mine) != 0;
        gang_retract(c, k);
        const double sum = block_sum(v);
        vmem_drain();
        return sum;
    });
    return o;
}

// ---------------------------------------------------------------------------
// out[i] = sum_j val[j] * v[col[j]] over the block's rows [r0, r1), each row
// summed in column-storage order (plain multiply, then add).  v may hold
// entries that other blocks wrote in this launch, so it is read with
// device-scope loads.
//
// A thread issues the gathers of its row's first SNZ entries before it adds.
// The matrix stays the same through the solve, so as many of the block's
// entries as fit are kept in LDS (the resident rows, the first n_res of the
// slice), and the first row per thread after them is loaded into registers
// before the barrier that completes v: of the three round trips of a row
// (bounds, entries, gathers) only the gathers are left behind the barrier.
// The rows after those are loaded a row ahead, their bounds two.  The entries
// past SNZ of long rows take their own round trips.
//
// Poisson 1024^2 (256 blocks of 1024 threads, 4096 rows each, half of them
// resident), per iteration with the two-pass qdot: 64 us with every entry
// read behind the barrier (the SpMV 20.5 of them), 66 with the products of
// coalesced entries staged through LDS, 53.7 with the resident rows; with the
// gathered sums 51.4, and 50.1 with the row ahead (this form spills 67 of its
// 128 VGPRs, 272 bytes of scratch per lane).  Two rows per thread in flight at
// once spilled more: 69.8.
// The batch of 24 systems (64 blocks of 256 threads for the largest, 4096
// rows each, a fifth of them resident): 4.66 ms, with the row ahead 3.82.
// ---------------------------------------------------------------------------
constexpr int SNZ = 8;

struct Bound {  // one row's entries
    int beg, len;
};

struct Row {  // bounds and first entries of one row
    Bound b;
    int ci[SNZ];
    double pv[SNZ];
};

// Row base + tid of the slice below r1 (empty past it).
__device__ __forceinline__ Bound load_bound(const CgSys &S, int64_t base, int64_t r1)
{
    const int64_t i = base + threadIdx.x;
    Bound b = {0, 0};
    if (i < r1) {
        b.beg = S.rowptr[i];
        b.len = S.rowptr[i + 1] - b.beg;
    }
    return b;
}

__device__ __forceinline__ void load_entries(const CgSys &S, Bound b, Row &R)
{
    R.b = b;
#pragma unroll
    for (int jj = 0; jj < SNZ; jj++) {
        R.ci[jj] = 0;
        R.pv[jj] = 0.0;
        if (jj < b.len) {
            R.ci[jj] = S.col[b.beg + jj];
            R.pv[jj] = S.val[b.beg + jj];
        }
    }
}

// What a thread holds of the rows after the resident ones before the barrier
// that completes v: the first row, and the next one's bounds.
struct RowsAhead {
    Row first;
    Bound next;
};

template <int NT>
__device__ __forceinline__ void load_ahead(const CgSys &S, int64_t base, int64_t r1, RowsAhead &R)
{
    load_entries(S, load_bound(S, base, r1), R.first);
    R.next = load_bound(S, base + NT, r1);
}

// The block's resident rows in LDS.
template <int NT, int LE>
struct MatLds {
    static constexpr int ROWS = LE / 2;  // resident rows at most
    double val[LE > 0 ? LE : 1];
    int col[LE > 0 ? LE : 1];
    unsigned short off[ROWS + 1];        // entries before row r0 + i
    int n_res;
};

template <int NT, int LE>
__device__ __forceinline__ void mat_load(const CgSys &S, int64_t r0, int64_t r1,
                                         MatLds<NT, LE> &M)
{
    static_assert(LE < 65536, "16-bit offsets");
    const int tid = threadIdx.x;
    if (tid == 0) M.n_res = 0;
    __syncthreads();
    if (r0 >= r1) return;
    const int e0 = S.rowptr[r0];
    const int ne = min(S.rowptr[r1] - e0, LE);
    for (int j = tid; j < ne; j += NT) {
        M.col[j] = S.col[e0 + j];
        M.val[j] = S.val[e0 + j];
    }
    const int nr = (int)min(r1 - r0, (int64_t)M.ROWS);
    int last = 0;
    for (int i = tid; i <= nr; i += NT) {
        const int o = S.rowptr[r0 + i] - e0;
        if (o <= LE) {
            M.off[i] = (unsigned short)o;
            last = i;  // rows below i are resident
        }
    }
    last = wave_reduce_i(last, [](int p, int q) { return max(p, q); });
    if ((tid & 63) == 0) atomicMax(&M.n_res, last);
    __syncthreads();
}

// R: load_ahead of the rows after the resident ones, taken before the barrier
// that completed v.  own(i, yi) is called once per row with its result.
template <int NT, int LE, class Own>
__device__ __forceinline__ void spmv_rows(const CgSys &S, const double *v, int64_t r0, int64_t r1,
                                          const MatLds<NT, LE> &M, RowsAhead &R, Own &&own)
{
    const int tid = threadIdx.x;
    const int n_res = M.n_res;
    for (int base = 0; base < n_res; base += NT) {
        const int i = base + tid;
        double g[SNZ];
        int beg = 0, len = 0;
        if (i < n_res) {
            beg = M.off[i];
            len = M.off[i + 1] - beg;
        }
#pragma unroll
        for (int jj = 0; jj < SNZ; jj++) {
            g[jj] = 0.0;
            if (jj < len) g[jj] = ld_dev(&v[M.col[beg + jj]]);
        }
        double s = 0.0;
#pragma unroll
        for (int jj = 0; jj < SNZ; jj++)
            if (jj < len) {
                const double pr = M.val[beg + jj] * g[jj];
                s = s + pr;
            }
        for (int j = beg + SNZ; j < beg + len; j++) {
            const double pr = M.val[j] * ld_dev(&v[M.col[j]]);
            s = s + pr;
        }
        if (i < n_res) own(r0 + i, s);
    }
    Row cur = R.first;
    Bound nb = R.next;
    for (int64_t base = r0 + n_res; base < r1; base += NT) {
        double g[SNZ];
#pragma unroll
        for (int jj = 0; jj < SNZ; jj++) {
            g[jj] = 0.0;
            if (jj < cur.b.len) g[jj] = ld_dev(&v[cur.ci[jj]]);
        }
        // the next row's entries, and the bounds after them, travel with the
        // gathers
        Row nxt;
        load_entries(S, nb, nxt);
        nb = load_bound(S, base + 2 * NT, r1);
        double s = 0.0;
#pragma unroll
        for (int jj = 0; jj < SNZ; jj++)
            if (jj < cur.b.len) {
                const double pr = cur.pv[jj] * g[jj];
                s = s + pr;
            }
        for (int j = cur.b.beg + SNZ; j < cur.b.beg + cur.b.len; j++) {
            const double pr = S.val[j] * ld_dev(&v[S.col[j]]);
            s = s + pr;
        }
        const int64_t i = base + tid;
        if (i < r1) own(i, s);
        cur = nxt;
    }
}

// One CG solve by one gang.
// ACC1: every inner product by the one-pass qdot (gang_qdot_s1, with the
// caller's LDS window S1 and the gang's table tab, 2 W S1_PIECES doubles);
// otherwise by the two-pass qdot, guaranteed with GUARD.
template <bool GUARD, int NT, int LE, bool ACC1 = false>
__device__ __forceinline__ void cg_solve(const CgSys &S, Gang *gg, int G, int gb, int key_mode,
                                         int score_mode, int nonstrict, CgLdsT<NT> &L,
                                         MatLds<NT, LE> &M,
                                         qdot_cg_result *res, S1Lds *S1 = nullptr,
                                         double *tab = nullptr)
{
    const int64_t n = S.n;
    // rows of this block: a multiple of CHUNK each, so qdot tiles line up
    const int64_t per = ((n + G - 1) / G + CHUNK - 1) / CHUNK * CHUNK;
    const int64_t r0 = min(n, (int64_t)gb * per), r1 = min(n, r0 + per);
    int k = 0;  // qdot buffer / partials parity
    int ntr = 0;
    GangCtx c = gang_enter(gg, G, gb);
    const SelArgs sa = {key_mode, score_mode, nonstrict, 0, S.qtol};
    auto dot = [&](const double *a, const double *bv, bool scanned = false, unsigned int sg = 0) {
        DotOut o;
        if (S.use_qdot) {
            qdot_result *ts = (gb == 0 && S.trace) ? S.trace + ntr : nullptr;
            if constexpr (ACC1)
                o = gang_qdot_s1(a, bv, n, r0, r1, S.qtol, key_mode, score_mode, nonstrict, c, k,
                                 L, *S1, tab + (size_t)k * W * S1_PIECES, ts);
            else
                o = gang_qdot<GUARD, NT>(a, bv, n, r0, r1, sa, c, k, L, ts, S.trace != nullptr,
                                         scanned, sg);
            ntr++;
        } else {
            o = gang_dot64<NT>(a, bv, r0, r1, c, k, L);
        }
        k ^= 1;
        return o;
    };
    int status = QDOT_OK, iters = 0;
    bool healthy = true;
    // r0 = b - A x0, p0 = r0
    mat_load<NT, LE>(S, r0, r1, M);
    RowsAhead R;
    load_ahead<NT>(S, r0 + M.n_res, r1, R);
    spmv_rows<NT, LE>(S, S.x, r0, r1, M, R, [&](int64_t i, double yi) {
        const double v = S.b[i] - yi;
        S.r[i] = v;
        st_dev(&S.p[i], v);
    });
    __syncthreads();
    DotOut bb = gang_dot64<NT>(S.b, S.b, r0, r1, c, k, L);
    k ^= 1;
    const double bnorm = sqrt(bb.value);
    const double thresh = S.rtol * bnorm;
    DotOut c0 = {0.0, false, false};
    if (bb.ok) c0 = dot(S.r, S.r);
    healthy = c0.ok;
    double rr = c0.value;
    bool done = false;
    if (healthy && c0.all_perf) {
        status = QDOT_E_BREAKDOWN;
        done = true;
    } else if (healthy && !(sqrt(rr) > thresh)) {
        done = true;
    }
    while (healthy && !done) {
        if (iters >= S.maxit) {
            status = QDOT_E_MAXIT;
            break;
        }
        load_ahead<NT>(S, r0 + M.n_res, r1, R);
        if (!(healthy = gang_barrier(c))) break;  // p complete
        // pass 1 of the two-pass qdot(p, q) rides in the SpMV; the one-pass
        // qdot reads its rows itself
        const bool scan_q = S.use_qdot != 0 && !ACC1;
        unsigned int sg1 = 0;
        spmv_rows<NT, LE>(S, S.p, r0, r1, M, R, [&](int64_t i, double yi) {
            S.q[i] = yi;
            if (scan_q) scan_pair(S.p[i], yi, key_mode, L.h, sg1);
        });
        __syncthreads();
        const DotOut d = dot(S.p, S.q, scan_q, sg1);
        if (!(healthy = d.ok)) break;
        if (!(d.value > 0.0) || !isfinite(d.value) || d.all_perf) {
            status = QDOT_E_BREAKDOWN;
            break;
        }
        const double alpha = rr / d.value;
        // x += alpha p, r -= alpha q (four rows' loads in flight per thread),
        // with pass 1 of the qdot r . r that follows fused in
        unsigned int sg2 = 0;
        const bool scan_r = S.use_qdot != 0 && !ACC1;
        auto xr_row = [&](int64_t i, double pi, double xi, double qi, double ri) {
            const double ap = alpha * pi;
            st_dev(&S.x[i], xi + ap);
            const double aq = alpha * qi;
            const double rn = ri - aq;
            S.r[i] = rn;
            if (scan_r) scan_pair(rn, rn, key_mode, L.h, sg2);
        };
        {
            int64_t i = r0 + threadIdx.x;
            for (; i + 3 * NT < r1; i += 4 * NT) {
                double pi[4], xi[4], qi[4], ri[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    pi[u] = S.p[i + u * NT];
                    xi[u] = S.x[i + u * NT];
                    qi[u] = S.q[i + u * NT];
                    ri[u] = S.r[i + u * NT];
                }
#pragma unroll
                for (int u = 0; u < 4; u++) xr_row(i + u * NT, pi[u], xi[u], qi[u], ri[u]);
            }
            for (; i < r1; i += NT) xr_row(i, S.p[i], S.x[i], S.q[i], S.r[i]);
        }
        __syncthreads();
        const DotOut cn = dot(S.r, S.r, scan_r, sg2);
        if (!(healthy = cn.ok)) break;
        if (cn.all_perf) {
            status = QDOT_E_BREAKDOWN;
            break;
        }
        const double beta = cn.value / rr;
        // p = r + beta p (four rows' loads in flight per thread)
        {
            int64_t i = r0 + threadIdx.x;
            for (; i + 3 * NT < r1; i += 4 * NT) {
                double pi[4], ri[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    pi[u] = S.p[i + u * NT];
                    ri[u] = S.r[i + u * NT];
                }
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const double bp = beta * pi[u];
                    st_dev(&S.p[i + u * NT], ri[u] + bp);
                }
            }
            for (; i < r1; i += NT) {
                const double bp = beta * S.p[i];
                st_dev(&S.p[i], S.r[i] + bp);
            }
        }
        rr = cn.value;
        iters++;
        if (!(sqrt(rr) > thresh)) done = true;
    }
    double relres_true = 0.0;
    if (healthy) healthy = gang_barrier(c);  // x complete
    if (healthy) {
        load_ahead<NT>(S, r0 + M.n_res, r1, R);
        spmv_rows<NT, LE>(S, S.x, r0, r1, M, R,
                          [&](int64_t i, double yi) { S.q[i] = S.b[i] - yi; });
        __syncthreads();
        const DotOut rq = gang_dot64<NT>(S.q, S.q, r0, r1, c, k, L);
        k ^= 1;
        healthy = rq.ok;
        relres_true = bnorm > 0.0 ? sqrt(rq.value) / bnorm : 0.0;
    }
    if (gb == 0 && threadIdx.x == 0) {
        res->iters = iters;
        res->status = healthy ? status : QDOT_E_DEVICE;
        res->relres_est = bnorm > 0.0 ? sqrt(rr) / bnorm : 0.0;
        res->relres_true = relres_true;
    }
    // leave the gang buffers clean and every block past its last use of them;
    // a gang that has given up leaves them to gang_reset, but this block's LDS
    // counts, of rows that were never merged, to nobody
    if (healthy)
        gang_barrier_then(c, [&] {
            if ((int)threadIdx.x < c.groups) {
                st_dev(&gg->val[0][threadIdx.x].w, NO_VALUE);
                st_dev(&gg->val[1][threadIdx.x].w, NO_VALUE);
            }
        });
    else
        for (int j = threadIdx.x; j < 4 * FQ; j += NT) L.h[j] = 0u;
    // the release is complete before this block enters the gang again
    vmem_drain();
    __syncthreads();
}

// Clears a gang's barrier, abort flag, values, partials and histogram buffers (plain
// stores; used by a kernel of its own, before the launch that uses the gang).
__device__ __forceinline__ void gang_reset(Gang *gg, unsigned int spin_limit,
                                           unsigned int join_spins = 0u)
{
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (int i = threadIdx.x; i < FQ; i += blockDim.x)
        for (int k = 0; k < 2; k++) {
            for (int q = 0; q < BAR_GROUPS; q++) gg->qb[k].hist[q][i] = z;
            gg->qb[k].hm[i] = z;
        }
    for (int k = 0; k < 2; k++)
        for (int i = threadIdx.x; i < MAX_GANG * 6; i += blockDim.x)
            gg->partials[k][i] = __longlong_as_double((long long)NO_VALUE);
    if (threadIdx.x < BAR_GROUPS) {
        gg->sub[threadIdx.x].v = 0u;
        gg->gen[threadIdx.x].v = 0u;
        gg->val[0][threadIdx.x].w = NO_VALUE;
        gg->val[1][threadIdx.x].w = NO_VALUE;
    }
    if (threadIdx.x == 0) {
        gg->join.v = 0u;
        gg->verdict.v = 0u;
        gg->top.v = 0u;
        gg->abort = 0u;
        gg->spin_limit = spin_limit;
        gg->join_spins = join_spins;
    }
}

}  // namespace qd
