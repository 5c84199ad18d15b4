// The two-pass qdot in two launches (any length), or in one (a length that
// one block holds in registers).
//
// k_key_scan counts the product exponents, as k_scan does.  k_sel_sweep is
// the selection, the sweep and the combine: every block reads the merged
// counts and selects the classes itself, into its own LDS table, sums its
// components, and the last block to finish adds up the blocks' sums, writes
// the whole result and clears the counts for the next call.  Nothing waits
// for another block, so the launches need no residency and no fence.
//
// A chain of four kernels (scan, selection, sweep, combine) is bound by
// latency until the vectors are long: on 1e5 components the selection alone,
// one workgroup of dependent loads and shuffle chains, took 8.4 us and the
// combine 4.1 us of 26.  Here the counts come in one round trip (whole
// histograms as 16-byte loads, without finding the live window first), the
// first group of operands is in flight meanwhile, and a block computes only
// what its sweep needs (e_max, t and the class of each live slot) before the
// sweep.  Counts, bound and flags are formed while the block's sums are on
// their way to memory, and only the last block uses them.  The start-up code
// runs once per block, so it is bound by instruction fetch: unrolled over the
// slots of a thread the selection took 1.4 us, as rolled loops over the live
// slots 0.4 us.
//
// Per call, back to back (four kernels -> here): 1000 components 20 -> 11 us
// (one block, 6.4 us in the kernel), 1e5 24.0 -> 13.8, 1e6 27.5 -> 18.0,
// guaranteed mode on 1e6 36.6 -> 20.9 (eight launches -> three), 1e7 72.4 ->
// 62.1.  Past 128 MiB per vector the guaranteed mode alone takes this form
// (the default mode below: k_spec_sweep).
//
// Classes, leaves and tile trees are those of the four-kernel chain, and so is
// the order of every FP64 sum where the launch shapes are the same (long
// vectors); on short vectors the compensated sums differ by the rounding of
// their error terms at most.
#include "qdot_kernels.hpp"

#include "qdot_guess.hpp"
#include "qdot_select.hpp"

namespace qd {

// A block's first group of NT * EPT * U components, loaded into registers
// ahead of the block's other start-up work.
template <bool VEC, int U, int NT, class T>
struct FirstGroup {
    T xv[U][4], yv[U][4];

    __device__ __forceinline__ static int lim_of(int64_t i0, int64_t n)
    {
        const int64_t left = n - i0;
        return left <= 0 ? 0 : (left >= 4 ? 4 : (int)left);
    }

    __device__ __forceinline__ void load(const T *__restrict__ x, const T *__restrict__ y,
                                         int64_t base, int64_t n)
    {
        constexpr int64_t chunk = (int64_t)NT * EPT;
        const bool full = base + chunk * U <= n;
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t i0 = base + u * chunk + threadIdx.x * EPT;
            if (full) {
                load4_full<VEC>(x + i0, xv[u]);
                load4_full<VEC>(y + i0, yv[u]);
            } else {
                load4_tail(x + i0, lim_of(i0, n), xv[u]);
                load4_tail(y + i0, lim_of(i0, n), yv[u]);
            }
        }
    }

    // body(xv, yv, lim) on each chunk; the whole group takes lim 4 as a
    // constant, so that its bounds tests fold away
    template <class Body>
    __device__ __forceinline__ void each(int64_t base, int64_t n, Body &&body) const
    {
        constexpr int64_t chunk = (int64_t)NT * EPT;
        if (base + chunk * U <= n) {
#pragma unroll
            for (int u = 0; u < U; u++) body(xv[u], yv[u], 4);
        } else {
#pragma unroll
            for (int u = 0; u < U; u++)
                body(xv[u], yv[u], lim_of(base + u * chunk + threadIdx.x * EPT, n));
        }
    }
};

// The block's counts into copy blockIdx % copies of dst: neighbouring lanes
// add to neighbouring slots, so that one request carries a line of them.
__device__ __forceinline__ void merge_counts(const unsigned int *h, uint4 (*dst)[FQ], int copies)
{
    unsigned int *gh = reinterpret_cast<unsigned int *>(dst[blockIdx.x % copies]);
    for (int i = threadIdx.x; i < 4 * FQ; i += BLOCK) {
        const unsigned int v = h[i];
        if (v) atomicAdd(&gh[i], v);
    }
}

// ---------------------------------------------------------------------------
// Pass 1: keys into the block's LDS histogram, merged into copy
// blockIdx % copies of the workspace's counts.
// ---------------------------------------------------------------------------
template <class T, bool VEC, int U>
__global__ __launch_bounds__(BLOCK) void k_key_scan(const T *__restrict__ x,
                                                    const T *__restrict__ y, int64_t n,
                                                    int key_mode, Ws *__restrict__ ws, int copies)
{
    __shared__ uint4 h4[FQ];
    unsigned int *h = reinterpret_cast<unsigned int *>(h4);
    const int64_t group = (int64_t)CHUNK * U;
    const int64_t stride = group * gridDim.x;
    const int64_t base = blockIdx.x * group;
    FirstGroup<VEC, U, BLOCK, T> g;
    g.load(x, y, base, n);
    for (int i = threadIdx.x; i < FQ; i += BLOCK) h4[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    unsigned int sg = 0;
    g.each(base, n, [&](const T *xv, const T *yv, int lim) { count4(xv, yv, lim, key_mode, h, sg); });
    stream_strided<VEC, U>(x, y, base + stride, stride, n,
                           [&](const T *xv, const T *yv, int64_t, int lim) {
                               count4(xv, yv, lim, key_mode, h, sg);
                           });
    count_signs(sg, h);
    __syncthreads();
    merge_counts(h, ws->fused.hist, copies);
}

// The power method's pair: x . w into wa and w . w into wb, x and w read once.
// On 128^3 components: 11.2 us here and 19.8 us in k_sel_sweep_pair, against
// 12.9 + 7.8 + 11.8 + 4.6 us in four kernels (80 -> 73 us per iteration).
template <bool VEC, int U>
__global__ __launch_bounds__(BLOCK) void k_key_scan_pair(const double *__restrict__ x,
                                                         const double *__restrict__ w, int64_t n,
                                                         int key_mode, Ws *__restrict__ wa,
                                                         Ws *__restrict__ wb, int copies)
{
    __shared__ uint4 h4[2 * FQ];
    unsigned int *ha = reinterpret_cast<unsigned int *>(h4);
    unsigned int *hb = reinterpret_cast<unsigned int *>(h4 + FQ);
    const int64_t group = (int64_t)CHUNK * U;
    const int64_t stride = group * gridDim.x;
    const int64_t base = blockIdx.x * group;
    FirstGroup<VEC, U, BLOCK, double> g;
    g.load(x, w, base, n);
    for (int i = threadIdx.x; i < 2 * FQ; i += BLOCK) h4[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    unsigned int sga = 0, sgb = 0;
    auto both = [&](const double *xv, const double *wv, int lim) {
        count4(xv, wv, lim, key_mode, ha, sga);
        count4(wv, wv, lim, key_mode, hb, sgb);
    };
    g.each(base, n, both);
    stream_strided<VEC, U>(
        x, w, base + stride, stride, n,
        [&](const double *xv, const double *wv, int64_t, int lim) { both(xv, wv, lim); });
    count_signs(sga, ha);
    count_signs(sgb, hb);
    __syncthreads();
    merge_counts(ha, wa->fused.hist, copies);
    merge_counts(hb, wb->fused.hist, copies);
}

// Counts this block as done with its sweep; true in every thread of the
// last of nblk blocks.  What the block stored before with device-scope
// stores is complete when it counts itself, so the last block sees it with
// device-scope loads.  Past 64 blocks they count in two levels, so that no
// counter takes more than nblk / 8 atomics in a row.  The counters are zero
// again afterwards.
__device__ __forceinline__ bool last_block(FusedWs &F, int blk, int nblk)
{
    __shared__ int s_last;
    if (threadIdx.x == 0) {
        vmem_drain();
        bool last = true;
        unsigned int all = (unsigned int)nblk;
        if (nblk > 64) {
            const int g = blk % ARRIVE_GROUPS;
            const unsigned int members =
                (unsigned int)((nblk - g + ARRIVE_GROUPS - 1) / ARRIVE_GROUPS);
            last = __hip_atomic_fetch_add(&F.sub[g][0], 1u, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) + 1 == members;
            if (last) st_dev(&F.sub[g][0], 0u);
            all = ARRIVE_GROUPS;
        }
        if (last)
            last = __hip_atomic_fetch_add(&F.arrive, 1u, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) + 1 == all;
        if (last) st_dev(&F.arrive, 0u);
        s_last = last;
    }
    __syncthreads();
    return s_last != 0;
}

// A block's sums: lanes 0..2 merge the waves' of one class each and store them
// (partials as six rows of nblk words, which the last block reads in whole
// lines).  A barrier precedes it.
__device__ __forceinline__ void store_partial(double *partials, int blk, int nblk,
                                              Acc (*red)[BLOCK / 64])
{
    const int q = threadIdx.x;
    if (q < 3) {
        Acc b = red[q][0];
#pragma unroll
        for (int w = 1; w < BLOCK / 64; w++) b = acc_merge(b, red[q][w]);
        st_dev(&partials[(size_t)(2 * q) * nblk + blk], b.s);
        st_dev(&partials[(size_t)(2 * q + 1) * nblk + blk], b.c);
    }
}

// The blocks' sums merged in a fixed order, per wave into red (a barrier has
// to follow).  Two blocks' sums are in flight per thread.
__device__ __forceinline__ void merge_partials(const double *partials, int nblk,
                                               Acc (*red)[BLOCK / 64])
{
    constexpr int P = 2;
    Acc f[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    for (int b0 = threadIdx.x; b0 < nblk; b0 += P * BLOCK) {
        Acc p[P][3];
#pragma unroll
        for (int u = 0; u < P; u++) {
            const int b = b0 + u * BLOCK;
#pragma unroll
            for (int q = 0; q < 3; q++) {
                p[u][q] = Acc{0.0, 0.0};
                if (b < nblk)
                    p[u][q] = Acc{ld_dev(&partials[(size_t)(2 * q) * nblk + b]),
                                  ld_dev(&partials[(size_t)(2 * q + 1) * nblk + b])};
            }
        }
#pragma unroll
        for (int u = 0; u < P; u++)
#pragma unroll
            for (int q = 0; q < 3; q++) f[q] = acc_merge(f[q], p[u][q]);
    }
    block_reduce3_waves<BLOCK, true>(f, red);
}

// ---------------------------------------------------------------------------
// Selection, sweep and combine of one product by blocks blk of nblk.
// GUARD (guard_mode 1): the last block also certifies the result, or selects
// the classes again and leaves them, the counts and g_redo to k_resweep.
// ---------------------------------------------------------------------------
// SPEC: after k_spec_sweep, whose counts are split over hist and samp (all
// copies); nothing is left to do when its guess stood.
template <class T, bool VEC, int U, bool GUARD, bool SPEC = false>
__device__ __forceinline__ void sel_sweep(const T *__restrict__ x, const T *__restrict__ y,
                                          int64_t n, const SelArgs &a, Ws *__restrict__ ws,
                                          int copies, double *__restrict__ partials,
                                          qdot_result *__restrict__ out, int blk, int nblk)
{
    constexpr int K = (FQ + BLOCK - 1) / BLOCK;
    __shared__ uint4 h4[FQ];
    __shared__ SelLds<BLOCK> S;
    __shared__ unsigned char lut[W_LUT];
    __shared__ Acc red[3][BLOCK / 64];
    __shared__ qdot_result R;
    const unsigned int *h = reinterpret_cast<const unsigned int *>(h4);
    const int tid = threadIdx.x;
    FusedWs &F = ws->fused;
    if (SPEC && F.done) return;

    uint4 v[K];
    {
        auto quad = [&](int c, int k) {
            const int q = k * BLOCK + tid;
            return q < FQ ? F.hist[0][c * FQ + q] : make_uint4(0u, 0u, 0u, 0u);
        };
        auto plus = [](uint4 p, uint4 r) {
            return make_uint4(p.x + r.x, p.y + r.y, p.z + r.z, p.w + r.w);
        };
        if constexpr (SPEC) {
            static_assert(offsetof(FusedWs, samp) == FH_COPIES * FQ * sizeof(uint4),
                          "samp follows hist");
#pragma unroll
            for (int k = 0; k < K; k++) v[k] = quad(0, k);
#pragma unroll 1
            for (int c = 1; c < (FH_COPIES + FS_COPIES); c++)
#pragma unroll
                for (int k = 0; k < K; k++) v[k] = plus(v[k], quad(c, k));
        } else if (copies == 1) {
#pragma unroll
            for (int k = 0; k < K; k++) v[k] = quad(0, k);
        } else {  // FH_COPIES (fused_copies)
            static_assert(FH_COPIES == 4, "four copies");
#pragma unroll
            for (int k = 0; k < K; k++)
                v[k] = plus(plus(quad(0, k), quad(1, k)), plus(quad(2, k), quad(3, k)));
        }
    }

    const int64_t group = (int64_t)CHUNK * U;
    const int64_t stride = group * nblk;
    const int64_t base = blk * group;
    FirstGroup<VEC, U, BLOCK, T> g;
    g.load(x, y, base, n);
    select_begin(S);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; k++)
        if (k * BLOCK + tid < FQ) h4[k * BLOCK + tid] = v[k];
    find_window<BLOCK, K>(v, S);
    __syncthreads();
    const Sel s = select_classes<BLOCK>(h, a, S, lut);
    Acc acc[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    if (s.live()) {
        auto leaves = [&](const T *xv, const T *yv, int lim) {
            acc_group<false>(xv, yv, lim, lut, a.key_mode, s.e_max, s.c32, true, acc[0], acc[1],
                             acc[2], nullptr);
        };
        g.each(base, n, leaves);
        stream_strided<VEC, U>(
            x, y, base + stride, stride, n,
            [&](const T *xv, const T *yv, int64_t, int lim) { leaves(xv, yv, lim); });
    }
    block_reduce3_waves<BLOCK, false>(acc, red);
    __syncthreads();
    store_partial(partials, blk, nblk, red);
    // only the last block needs them; here they cost it nothing, while its
    // sums are on their way to memory
    select_count<BLOCK>(h, s, a, S);
    if (!last_block(F, blk, nblk)) return;

    // the last block: the result, and the counts zero for the next call
    merge_partials(partials, nblk, red);
    for (int i = tid; i < (SPEC ? (FH_COPIES + FS_COPIES) : copies) * FQ; i += BLOCK)
        F.hist[0][i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    finish_result<BLOCK>(s, a, n, S, red, R);
    if constexpr (GUARD) {
        __shared__ int s_dref;
        const int lo = s.n_bins ? s.e_min - KMIN : W, hi = s.n_bins ? s.e_max - KMIN : -1;
        const bool go = s.live();
        GuardSums gs = {0.0, 0.0, 0.0};
        if (go) gs = guard_sums<BLOCK>([&](int j) { return h[j]; }, lut, lo, hi, s.e_max);
        if (tid == 0) {
            s_dref = 0;
            ws->g_redo = 0;
            // every product zero: +0 is exact
            if (s.status == QDOT_OK && s.n_bins == 0) R.flags |= QDOT_F_GUARANTEED;
            if (go) {
                const double low = guard_lower(gs, S.sum, n, s.signs);
                if (guard_certified(R.bound_rel, low, a.tol)) {
                    R.flags |= QDOT_F_GUARANTEED;
                    R.lower = ldexp(low, s.e_max);
                } else {
                    // L <= 0: every bin at the input precision (scores >= 23
                    // for double inputs, >= 10 for single; one more
                    // non-strict)
                    const int ref = low > 0.0 ? s.e_max + ilogb(low)
                                              : s.e_min - s.t - (a.mu_single ? 9 : 22) - a.nonstrict;
                    if (ref < s.e_max) {
                        s_dref = s.e_max - ref;
                        ws->g_low = low;
                        ws->g_redo = 1;
                    } else {
                        R.lower = low > 0.0 ? ldexp(low, s.e_max) : 0.0;
                    }
                }
            }
        }
        __syncthreads();
        if (s_dref) {
            const int passes = R.passes;
            __syncthreads();
            // k_resweep certifies with the same counts
            for (int j = lo + tid; j <= hi; j += BLOCK) ws->hsave[j] = h[j];
            auto get = [&](int j) { return (unsigned long long)h[j]; };
            auto put = [&](int j, int cls) { ws->lut[j] = (unsigned char)cls; };
            auto clear = [](int) {};
            const CutParams p =
                block_cutoff<BLOCK>(lo, hi, s.n_zero, 0u, n, a.tol, a.score_mode, a.nonstrict,
                                    get, put, clear, &R, nullptr, s_dref, a.mu_single);
            if (tid < W_LUT - W) ws->lut[W + tid] = (unsigned char)QDOT_PERF;
            if (tid == 0) {
                ws->e_max = s.e_max;
                ws->c32 = p.c32;
                ws->flags = p.flags | QDOT_F_RESELECTED;
                ws->skip = p.skip;
                ws->s1_lo = lo;
                ws->s1_hi = hi;
                ws->signs = s.signs;
                R.flags |= QDOT_F_RESELECTED;
                R.passes = passes + (p.skip ? 0 : 1);
            }
        }
    }
    __syncthreads();
    put_result(out, R);
}

template <class T, bool VEC, int U, bool GUARD, bool SPEC = false>
__global__ __launch_bounds__(BLOCK, GUARD ? 1 : 4) void k_sel_sweep(const T *__restrict__ x,
                                                     const T *__restrict__ y, int64_t n,
                                                     SelArgs a, Ws *__restrict__ ws, int copies,
                                                     double *__restrict__ partials,
                                                     qdot_result *__restrict__ out)
{
    sel_sweep<T, VEC, U, GUARD, SPEC>(x, y, n, a, ws, copies, partials, out, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// Long vectors, one pass over them where it can be: k_key_sample counts a
// sample (one run in 2^up), every block of k_spec_sweep selects the classes from
// the sample's counts as if they were the whole's, and reads its components
// once, counting them and summing their leaves by the guessed classes.  The
// last block selects from the whole counts: when every live bin has the class
// that was guessed, the sums are those of the sweep, and it writes the result.
// When one has not, k_sel_sweep sums again with the right classes: the counts
// are complete, so nothing but time is lost.  The guess enters no result.
//
// The guess stands when the sample sees the largest exponent and no count
// near a class boundary lies within its error of a power of two.  Where that
// is not likely (guess_holds) k_spec_sweep only counts, and k_sel_sweep sums as
// always.
//
// The bound is HBM: 16 bytes per component once, plus the sample again, in
// place of twice 16.  2^27 components: 699 us with two passes, 381 where the
// guess stands (10**U[-20, 20], family A), 700 where it is not used (normal,
// uniform, family B).  5e7 floats: 168, 121 and 170.
// Left to the blocks of one scan, which started to sum once the sample was
// counted, it took 475 us: the guess came 25 us into the launch.
// ---------------------------------------------------------------------------

// Words of guess_holds in LDS: `dense` W and the others zero before it, with
// a barrier between.
struct GuessLds {
    int dense;  // the lowest slot that the sample saw GUESS_SEEN times
    int empty;  // empty slots of the window below it
    int risk;   // sum of slot_risk
};

// Whether to sum by the classes that the sample's counts h (scaled by 2^up)
// select (s, from them): top_holds, t is the same with the rare bins that the
// sample did not see, and the slots' risks sum to GUESS_RISK at most.  Every
// thread of the block calls it, after a barrier, and gets the same answer,
// which is the same in every block: the risks are whole numbers.
__device__ __forceinline__ bool guess_holds(const unsigned int *h, const Sel &s,
                                            const SelArgs &a, int up, GuessLds &G)
{
    if (!s.live()) return false;
    const int tid = threadIdx.x, lane = tid & 63;
    const int bot = s.e_min - KMIN, top = s.e_max - KMIN;
    if (!top_holds(h, top, up)) return false;
    int dense = W;
#pragma unroll 1
    for (int j = bot + tid; j <= top && dense == W; j += BLOCK)
        if (h[j] >= GUESS_SEEN) dense = j;
    dense = wave_reduce_i(dense, [](int p, int r) { return min(p, r); });
    if (lane == 0) atomicMin(&G.dense, dense);
    __syncthreads();
    dense = G.dense;
    int empty = 0, risk = 0;
#pragma unroll 1
    for (int j = bot - 1 + tid; j <= top; j += BLOCK) {
        const unsigned int m = j < bot ? 0u : h[j];
        if (m == 0u && !(j < dense && bot < dense)) continue;
        empty += m == 0u && j >= bot;
        const int base = j + KMIN - s.e_max - s.t + 1;  // the score of a count of 1
        risk += slot_risk(m, sigma_of(m, j, s) - base, base + up, a.nonstrict, a.mu_single);
    }
    auto add = [](int p, int r) { return p + r; };
    empty = wave_reduce_i(empty, add);
    risk = wave_reduce_i(risk, add);
    if (lane == 0) {
        atomicAdd(&G.empty, empty);
        atomicAdd(&G.risk, risk);
    }
    __syncthreads();
    if (a.score_mode == 0 && bot < dense &&
        floor_log2_ratio(a.tol, (unsigned long long)(s.n_bins + G.empty + up + 2)) != s.t)
        return false;
    return G.risk <= GUESS_RISK;
}

// Runs of 4 CHUNK components; the multiples of 2^up are the sample.
constexpr int64_t SAMPLE_RUN = 4 * CHUNK;

// Counts the groups of CHUNK * U components of the runs that run(j) gives for
// j = 0, 1, ..., below `runs`, block by block.
template <class T, bool VEC, int U, class Run>
__device__ __forceinline__ void count_runs(const T *__restrict__ x, const T *__restrict__ y,
                                           int64_t n, int key_mode, unsigned int *h, Run &&run)
{
    constexpr unsigned int PER = 4 / U;  // groups of a run
    const unsigned int runs = (unsigned int)((n + SAMPLE_RUN - 1) / SAMPLE_RUN);
    const int64_t past = n + SAMPLE_RUN;  // a stride that ends the walk
    unsigned int signs = 0;  // not needed here: no guard follows
    for (unsigned int i = blockIdx.x;; i += gridDim.x) {
        const unsigned int r = run(i / PER);
        if (r >= runs) break;
        stream_strided<VEC, U>(x, y, r * SAMPLE_RUN + (i % PER) * ((int64_t)CHUNK * U), past, n,
                               [&](const T *xv, const T *yv, int64_t, int lim) {
                                   count4(xv, yv, lim, key_mode, h, signs);
                               });
    }
}

template <class T, bool VEC>
__global__ __launch_bounds__(BLOCK) void k_key_sample(const T *__restrict__ x,
                                                      const T *__restrict__ y, int64_t n,
                                                      int key_mode, Ws *__restrict__ ws, int up)
{
    __shared__ uint4 h4[FQ];
    unsigned int *h = reinterpret_cast<unsigned int *>(h4);
    // the last block of k_spec_sweep alone sets it: two blocks of one launch
    // must not store the same word, as their L2s write back in any order
    if (blockIdx.x == 0 && threadIdx.x == 0) ws->fused.done = 0;
    for (int i = threadIdx.x; i < FQ; i += BLOCK) h4[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    count_runs<T, VEC, 4>(x, y, n, key_mode, h, [&](unsigned int j) { return j << up; });
    __syncthreads();
    merge_counts(h, ws->fused.samp, FS_COPIES);
}

template <class T, bool VEC, int U>
__global__ __launch_bounds__(BLOCK, 4) void k_spec_sweep(const T *__restrict__ x,
                                                         const T *__restrict__ y, int64_t n,
                                                         SelArgs a, Ws *__restrict__ ws, int up,
                                                         double *__restrict__ partials,
                                                         qdot_result *__restrict__ out)
{
    constexpr int K = (FQ + BLOCK - 1) / BLOCK;
    __shared__ uint4 h4[FQ];
    __shared__ SelLds<BLOCK> S;
    __shared__ unsigned int lut32[W_LUT / 4];
    __shared__ Acc red[3][BLOCK / 64];
    __shared__ qdot_result R;
    __shared__ int s_miss;
    __shared__ GuessLds G;
    unsigned int *h = reinterpret_cast<unsigned int *>(h4);
    unsigned char *lut = reinterpret_cast<unsigned char *>(lut32);
    const int tid = threadIdx.x;
    FusedWs &F = ws->fused;
    const uint4 z4 = make_uint4(0u, 0u, 0u, 0u);
    auto plus = [](uint4 p, uint4 r) {
        return make_uint4(p.x + r.x, p.y + r.y, p.z + r.z, p.w + r.w);
    };
    // a window of counts (v) into LDS, ready for select_classes
    auto to_lds = [&](const uint4 (&v)[K]) {
        select_begin(S);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; k++)
            if (k * BLOCK + tid < FQ) h4[k * BLOCK + tid] = v[k];
        find_window<BLOCK, K>(v, S);
        __syncthreads();
    };

    // the guess; slots that the sample did not see are perforated
    bool sum;
    Sel g;
    {
        uint4 v[K];
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int q = k * BLOCK + tid;
            v[k] = z4;
            if (q < FQ)
                for (int c = 0; c < FS_COPIES; c++) v[k] = plus(v[k], F.samp[c][q]);
        }
        for (int i = tid; i < W_LUT / 4; i += BLOCK) lut32[i] = 0x01010101u * QDOT_PERF;
        if (tid == 0) G = GuessLds{W, 0, 0};
        to_lds(v);
        g = select_classes<BLOCK>(h, a, S, lut, up);
        sum = guess_holds(h, g, a, up, G);
        __syncthreads();
        for (int i = tid; i < FQ; i += BLOCK) h4[i] = z4;
        __syncthreads();
    }

    if (!sum) {
        // the scan's own shape (one group of doubles in flight, two of floats)
        const unsigned int rest = (1u << up) - 1u;  // runs after each one of the sample
        count_runs<T, VEC, sizeof(T) == 4 ? 2 : 1>(
            x, y, n, a.key_mode, h,
            [&](unsigned int j) { return j / rest * (rest + 1u) + j % rest + 1u; });
        __syncthreads();
        merge_counts(h, F.hist, FH_COPIES);
        return;
    }
    const int64_t group = (int64_t)CHUNK * U;
    const int64_t past = n + group;  // a stride that ends the walk
    Acc acc[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    for (unsigned int i = blockIdx.x; i * group < n; i += gridDim.x) {
        const bool count = ((i / (unsigned)(4 / U)) & ((1u << up) - 1u)) != 0u;  // not yet counted
        stream_strided<VEC, U>(x, y, i * group, past, n,
                               [&](const T *xv, const T *yv, int64_t, int lim) {
                                   acc_group<false, true>(xv, yv, lim, lut, a.key_mode, g.e_max,
                                                          g.c32, true, acc[0], acc[1], acc[2],
                                                          nullptr, h, count);
                               });
    }
    block_reduce3_waves<BLOCK, false>(acc, red);
    __syncthreads();
    merge_counts(h, F.hist, FH_COPIES);
    store_partial(partials, blockIdx.x, gridDim.x, red);
    vmem_drain();
    __syncthreads();
    if (!last_block(F, blockIdx.x, gridDim.x)) return;

    if (tid == 0) s_miss = 0;
    // the whole counts
    uint4 v[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int q = k * BLOCK + tid;
        v[k] = z4;
        if (q < FQ)
            for (int c = 0; c < (FH_COPIES + FS_COPIES); c++) v[k] = plus(v[k], ld_dev_quad(&F.hist[0][c * FQ + q]));
    }
    to_lds(v);
    __shared__ unsigned char lut2[W_LUT];
    const Sel s = select_classes<BLOCK>(h, a, S, lut2);
    if (s.live())
        for (int j = s.e_min - KMIN + tid; j <= s.e_max - KMIN; j += BLOCK)
            if (h[j] && lut2[j] != lut[j]) s_miss = 1;
    // FP32 leaves stay far inside their range in the guess's units too
    if (tid == 0 && (!s.live() || abs(s.c32 - g.c32) > 32 || abs(s.e_max - g.e_max) > 32))
        s_miss = 1;
    merge_partials(partials, gridDim.x, red);
    select_count<BLOCK>(h, s, a, S);
    __syncthreads();
    if (s_miss) return;
    for (int i = tid; i < (FH_COPIES + FS_COPIES) * FQ; i += BLOCK) F.hist[0][i] = z4;
    finish_result<BLOCK>(s, a, n, S, red, R, g.e_max, g.c32);
    put_result(out, R);
    if (tid == 0) F.done = 1;
}

// The power method's pair in one grid of 2 g blocks: x . w (wa) in the first
// half, w . w (wb) in the second, each with its own counters.
template <bool VEC, int U, bool GUARD>
__global__ __launch_bounds__(BLOCK, GUARD ? 1 : 4) void k_sel_sweep_pair(
    const double *__restrict__ x, const double *__restrict__ w, int64_t n, SelArgs a,
    Ws *__restrict__ wa, Ws *__restrict__ wb, int copies, double *__restrict__ partials,
    qdot_result *__restrict__ out_a, qdot_result *__restrict__ out_b, int g)
{
    const bool first = (int)blockIdx.x < g;
    sel_sweep<double, VEC, U, GUARD>(first ? x : w, w, n, a, first ? wa : wb, copies,
                                     first ? partials : partials + (size_t)6 * g,
                                     first ? out_a : out_b,
                                     first ? (int)blockIdx.x : (int)blockIdx.x - g, g);
}

// Guaranteed mode, after a reselection (g_redo): the second sweep with the
// classes in the workspace, its combine, and the check with the larger lower
// bound.  Returns at once when the first selection stood.
template <class T, bool VEC, int U>
__global__ __launch_bounds__(BLOCK) void k_resweep(const T *__restrict__ x,
                                                   const T *__restrict__ y, int64_t n,
                                                   SelArgs a, Ws *__restrict__ ws,
                                                   double *__restrict__ partials,
                                                   qdot_result *__restrict__ out)
{
    __shared__ unsigned int lut32[W_LUT / 4];
    __shared__ Acc red[3][BLOCK / 64];
    __shared__ qdot_result R;
    if (!ws->g_redo) return;
    const unsigned char *lut = reinterpret_cast<const unsigned char *>(lut32);
    const int tid = threadIdx.x;
    const int e_max = ws->e_max, c32 = ws->c32, skip = ws->skip;
    for (int i = tid; i < W_LUT / 4; i += BLOCK)
        lut32[i] = reinterpret_cast<const unsigned int *>(ws->lut)[i];
    __syncthreads();
    Acc acc[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
    if (!skip)
        stream_groups<VEC, U>(x, y, n, [&](const T *xv, const T *yv, int64_t, int lim) {
            acc_group<false>(xv, yv, lim, lut, a.key_mode, e_max, c32, true, acc[0], acc[1],
                             acc[2], nullptr);
        });
    block_reduce3_waves<BLOCK, false>(acc, red);
    __syncthreads();
    store_partial(partials, blockIdx.x, gridDim.x, red);
    if (!last_block(ws->fused, blockIdx.x, gridDim.x)) return;
    merge_partials(partials, gridDim.x, red);
    const GuardSums g = guard_sums<BLOCK>([&](int j) { return ws->hsave[j]; }, lut, ws->s1_lo,
                                          ws->s1_hi, e_max);
    __syncthreads();
    if (tid == 0) {
        R = *out;
        Acc f[3];
        for (int q = 0; q < 3; q++) {
            f[q] = red[q][0];
            for (int w = 1; w < BLOCK / 64; w++) f[q] = acc_merge(f[q], red[q][w]);
        }
        const double sum =
            skip ? 0.0 : combine_value(f, e_max, c32, ws->flags, &R, a.mu_single);
        const double low = fmax(guard_lower(g, sum, n, ws->signs), ws->g_low);
        R.flags |= QDOT_F_RESELECTED |
                   (guard_certified(R.bound_rel, low, a.tol) ? QDOT_F_GUARANTEED : 0);
        R.lower = low > 0.0 ? ldexp(low, e_max) : 0.0;
    }
    __syncthreads();
    put_result(out, R);
}

// ---------------------------------------------------------------------------
// The whole qdot by one block that keeps its components in registers: n <=
// 4 NT U.
// ---------------------------------------------------------------------------
template <class T, bool VEC, int U, int NT, bool GUARD>
__global__ __launch_bounds__(NT) void k_qdot_block(const T *__restrict__ x,
                                                   const T *__restrict__ y, int64_t n,
                                                   SelArgs a, qdot_result *__restrict__ out)
{
    constexpr int K = (FQ + NT - 1) / NT;
    __shared__ uint4 h4[FQ];
    __shared__ SelLds<NT> S;
    __shared__ unsigned char lut[W_LUT];
    __shared__ Acc red[3][NT / 64];
    __shared__ qdot_result R;
    unsigned int *h = reinterpret_cast<unsigned int *>(h4);
    const int tid = threadIdx.x;
    FirstGroup<VEC, U, NT, T> g;
    g.load(x, y, 0, n);
    for (int i = tid; i < FQ; i += NT) h4[i] = make_uint4(0u, 0u, 0u, 0u);
    select_begin(S);
    __syncthreads();
    unsigned int sg = 0;
    g.each(0, n, [&](const T *xv, const T *yv, int lim) { count4(xv, yv, lim, a.key_mode, h, sg); });
    count_signs(sg, h);
    __syncthreads();
    uint4 v[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int q = k * NT + tid;
        v[k] = q < FQ ? h4[q] : make_uint4(0u, 0u, 0u, 0u);
    }
    find_window<NT, K>(v, S);
    __syncthreads();
    const Sel s = select_classes<NT>(h, a, S, lut);
    auto sweep = [&](int e_max, int c32, Acc acc[3]) {
        for (int q = 0; q < 3; q++) acc[q] = Acc{0.0, 0.0};
        g.each(0, n, [&](const T *xv, const T *yv, int lim) {
            acc_group<false>(xv, yv, lim, lut, a.key_mode, e_max, c32, true, acc[0], acc[1],
                             acc[2], nullptr);
        });
        block_reduce3_waves<NT, false>(acc, red);
        __syncthreads();
    };
    Acc acc[3];
    select_count<NT>(h, s, a, S);
    if (s.live()) sweep(s.e_max, s.c32, acc);
    else __syncthreads();
    finish_result<NT>(s, a, n, S, red, R);
    if constexpr (GUARD) {
        const int lo = s.n_bins ? s.e_min - KMIN : W, hi = s.n_bins ? s.e_max - KMIN : -1;
        auto get = [&](int j) { return (unsigned long long)h[j]; };
        auto put = [&](int j, int c) { lut[j] = (unsigned char)c; };
        block_guard<NT>(
            lo, hi, s.n_zero, s.signs, n, a.tol, a.score_mode, a.nonstrict, get, put, lut, S.sum, R,
            [&](const CutParams &p, int flags) {
                Acc b[3];
                sweep(p.e_max, p.c32, b);
                if (tid != 0) return 0.0;
                for (int q = 0; q < 3; q++) {
                    b[q] = red[q][0];
                    for (int w = 1; w < NT / 64; w++) b[q] = acc_merge(b[q], red[q][w]);
                }
                return combine_value(b, p.e_max, p.c32, flags, &R, a.mu_single);
            },
            a.mu_single);
    }
    __syncthreads();
    put_result(out, R);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
template <int U>
static int fused_grid(int64_t n, int cap)
{
    const int64_t groups = (n + (int64_t)CHUNK * U - 1) / ((int64_t)CHUNK * U);
    return (int)std::max<int64_t>(1, std::min<int64_t>(cap, groups));
}

// Copies of the counts that the scan's blocks spread over: the adds of one
// slot queue at its address, and every block of the sweep reads every copy.
// On 98 blocks 2 and 4 copies took the same time, on 256 to 512 four were
// 0.5 to 2 us faster than two.
static int fused_copies(int grid) { return grid <= 64 ? 1 : FH_COPIES; }

// Pass 1; returns the copies of the counts that it used.
template <class T, bool VEC, int U>
static int launch_key_scan(const Launch &L, const T *x, const T *y, int64_t n, int key_mode)
{
    const int grid = fused_grid<U>(n, L.scan_blocks), copies = fused_copies(grid);
    hipLaunchKernelGGL((k_key_scan<T, VEC, U>), dim3(grid), dim3(BLOCK), 0, L.stream, x, y, n,
                       key_mode, L.ws, copies);
    return copies;
}

template <class T, bool VEC, int U>
static void launch_sel_sweep(const Launch &L, const T *x, const T *y, int64_t n,
                             const SelArgs &a, int copies, int guard, qdot_result *out)
{
    const dim3 grid(fused_grid<U>(n, L.acc_blocks));
    if (guard) {
        hipLaunchKernelGGL((k_sel_sweep<T, VEC, U, true>), grid, dim3(BLOCK), 0, L.stream, x, y,
                           n, a, L.ws, copies, L.partials, out);
        hipLaunchKernelGGL((k_resweep<T, VEC, U>), grid, dim3(BLOCK), 0, L.stream, x, y, n, a,
                           L.ws, L.partials, out);
    } else {
        hipLaunchKernelGGL((k_sel_sweep<T, VEC, U, false>), grid, dim3(BLOCK), 0, L.stream, x, y,
                           n, a, L.ws, copies, L.partials, out);
    }
}


// The sample, the sweep by the guessed classes, and the scan and sweep of a
// call whose guess was not taken or did not stand.
template <class T, bool VEC>
static void launch_spec(const Launch &L, const T *x, const T *y, int64_t n, const SelArgs &a,
                        int up, qdot_result *out)
{
    // groups in flight: four of floats while counting too, two in the sweep,
    // whose four would spill
    constexpr int U = sizeof(T) == 4 ? 4 : 2;
    const int grid = fused_grid<U>(n, L.acc_blocks);
    hipLaunchKernelGGL((k_key_sample<T, VEC>), dim3(fused_grid<4>(n >> up, 512)), dim3(BLOCK), 0,
                       L.stream, x, y, n, a.key_mode, L.ws, up);
    if (L.ev) {
        (void)hipEventRecord(L.ev[1], L.stream);
        (void)hipEventRecord(L.ev[2], L.stream);
    }
    hipLaunchKernelGGL((k_spec_sweep<T, VEC, U>), dim3(grid), dim3(BLOCK), 0, L.stream, x, y, n, a,
                       L.ws, up, L.partials, out);
    // returns at once when the guess stood
    hipLaunchKernelGGL((k_sel_sweep<T, VEC, 2, false, true>), dim3(grid), dim3(BLOCK), 0, L.stream,
                       x, y, n, a, L.ws, FH_COPIES, L.partials, out);
}

template <class T, bool VEC, int U, int NT>
static void launch_block_u(const Launch &L, const T *x, const T *y, int64_t n,
                           const SelArgs &a, int guard, qdot_result *out)
{
    if (guard)
        hipLaunchKernelGGL((k_qdot_block<T, VEC, U, NT, true>), dim3(1), dim3(NT), 0, L.stream, x,
                           y, n, a, out);
    else
        hipLaunchKernelGGL((k_qdot_block<T, VEC, U, NT, false>), dim3(1), dim3(NT), 0, L.stream, x,
                           y, n, a, out);
}

// One block takes a vector of one group of 1024 threads: on 4000 components
// it took 11.6 us against 14.2 in two launches (and 11.5 against 20.3 in four
// on 1000); on 8000, two groups, 17.1 against 14.2, one CU's arithmetic.
constexpr int64_t ONE_BLOCK_MAX = 4096;
// Up to this length every chunk gets a block of its own: on 3e5 components
// 15.7 us, against 17.5 with four chunks per block in flight (floats 16.3
// against 22.5).
constexpr int64_t WIDE_MAX = (int64_t)CHUNK * 512;

// The sweep by guessed classes from 128 MiB per vector, where both no longer
// fit the memory-side cache: there a guess that is not used costs what the
// sample's launch does (2^24 normal products 97 us against 92, 2^27 700
// against 687), and one that stands saves a pass.  A wrong one costs the sums
// made for it (5e7 products 309 us, 172 when it stands).  The sample has at
// least SPEC_SAMPLE components, less than twice that: the top bin of
// 10**U[-20, 20] products then holds 91 or more.  On 24 draws each at 5e7
// (three tolerances, by the top and t alone), 5 * 2^19 components guessed 21
// rightly, 2^22 and 2^23 components 23, and 2^23 took 15 us more.
constexpr int64_t SPEC_MIN_BYTES = (int64_t)1 << 27;
constexpr int64_t SPEC_SAMPLE = (int64_t)1 << 22;

template <class T, bool VEC>
static void launch_fused_v(const Launch &L, const T *x, const T *y, int64_t n,
                           const SelArgs &a, int guard, qdot_result *out)
{
    if (n <= ONE_BLOCK_MAX) {
        if (n <= 1024) launch_block_u<T, VEC, 1, 256>(L, x, y, n, a, guard, out);
        else launch_block_u<T, VEC, 1, 1024>(L, x, y, n, a, guard, out);
        if (L.ev) {
            (void)hipEventRecord(L.ev[1], L.stream);
            (void)hipEventRecord(L.ev[2], L.stream);
        }
        return;
    }
    if (n * (int64_t)sizeof(T) >= SPEC_MIN_BYTES && !guard) {
        int up = 2;
        while ((n >> (up + 1)) >= SPEC_SAMPLE) up++;
        return launch_spec<T, VEC>(L, x, y, n, a, up, out);
    }
    // longer vectors take the tuned groups in flight (twice as many for floats)
    const int f = sizeof(T) == 4 ? 2 : 1;
    const bool wide = n <= WIDE_MAX;
    const int us = wide ? 1 : std::min(4, f * L.scan_unroll);
    const int ua = wide ? 1 : std::min(4, f * L.acc_unroll);
    const int copies = us == 1   ? launch_key_scan<T, VEC, 1>(L, x, y, n, a.key_mode)
                       : us == 2 ? launch_key_scan<T, VEC, 2>(L, x, y, n, a.key_mode)
                                 : launch_key_scan<T, VEC, 4>(L, x, y, n, a.key_mode);
    if (L.ev) {
        (void)hipEventRecord(L.ev[1], L.stream);
        (void)hipEventRecord(L.ev[2], L.stream);
    }
    // (four groups of doubles ahead of the selection would spill)
    if (ua == 1) launch_sel_sweep<T, VEC, 1>(L, x, y, n, a, copies, guard, out);
    else if (ua == 2 || sizeof(T) == 8)
        launch_sel_sweep<T, VEC, 2>(L, x, y, n, a, copies, guard, out);
    else if constexpr (sizeof(T) == 4)
        launch_sel_sweep<T, VEC, 4>(L, x, y, n, a, copies, guard, out);
}

template <class T>
static hipError_t launch_fused_t(const Launch &L, const T *x, const T *y, int64_t n, double tol,
                                 const qdot_options &o, qdot_result *out)
{
    const bool vec = ((((uintptr_t)x) | ((uintptr_t)y)) & 15) == 0;
    const SelArgs a = {o.key_mode, o.score_mode, o.boundary_mode, sizeof(T) == 4 ? 1 : 0, tol};
    if (L.ev) (void)hipEventRecord(L.ev[0], L.stream);
    if (vec) launch_fused_v<T, true>(L, x, y, n, a, o.guard_mode, out);
    else launch_fused_v<T, false>(L, x, y, n, a, o.guard_mode, out);
    if (L.ev) {
        (void)hipEventRecord(L.ev[3], L.stream);
        (void)hipEventRecord(L.ev[4], L.stream);
    }
    return hipGetLastError();
}

template <bool VEC, int U>
static void launch_pair_u(const Launch &La, const Launch &Lb, const double *x, const double *w,
                          int64_t n, const SelArgs &a, int guard, qdot_result *out_a,
                          qdot_result *out_b)
{
    hipStream_t s = La.stream;
    const int gs = fused_grid<U>(n, La.scan_blocks), copies = fused_copies(gs);
    const int g = std::min(fused_grid<U>(n, La.acc_blocks), La.partial_cap / 2);
    hipLaunchKernelGGL((k_key_scan_pair<VEC, U>), dim3(gs), dim3(BLOCK), 0, s, x, w, n,
                       a.key_mode, La.ws, Lb.ws, copies);
    if (guard) {
        hipLaunchKernelGGL((k_sel_sweep_pair<VEC, U, true>), dim3(2 * g), dim3(BLOCK), 0, s, x, w,
                           n, a, La.ws, Lb.ws, copies, La.partials, out_a, out_b, g);
        hipLaunchKernelGGL((k_resweep<double, VEC, U>), dim3(g), dim3(BLOCK), 0, s, x, w, n, a,
                           La.ws, La.partials, out_a);
        hipLaunchKernelGGL((k_resweep<double, VEC, U>), dim3(g), dim3(BLOCK), 0, s, w, w, n, a,
                           Lb.ws, La.partials, out_b);
    } else {
        hipLaunchKernelGGL((k_sel_sweep_pair<VEC, U, false>), dim3(2 * g), dim3(BLOCK), 0, s, x,
                           w, n, a, La.ws, Lb.ws, copies, La.partials, out_a, out_b, g);
    }
}

hipError_t launch_fused_pair(const Launch &La, const Launch &Lb, const double *x,
                             const double *w, int64_t n, double tol, const qdot_options &o,
                             qdot_result *out_a, qdot_result *out_b)
{
    const bool vec = ((((uintptr_t)x) | ((uintptr_t)w)) & 15) == 0;
    const SelArgs a = {o.key_mode, o.score_mode, o.boundary_mode, 0, tol};
    const bool one = n <= WIDE_MAX || La.acc_unroll == 1;
    if (vec && one) launch_pair_u<true, 1>(La, Lb, x, w, n, a, o.guard_mode, out_a, out_b);
    else if (vec) launch_pair_u<true, 2>(La, Lb, x, w, n, a, o.guard_mode, out_a, out_b);
    else launch_pair_u<false, 1>(La, Lb, x, w, n, a, o.guard_mode, out_a, out_b);
    return hipGetLastError();
}

bool fused_ok(const Launch &L, int64_t n, const qdot_options &o)
{
    // 32-bit counts; the tuned variants of the four-kernel chain (threads per
    // block, compacting sweep) and its other selections stay there.  Tile keys
    // save reads, which bound long vectors only: on 2^20 components the chain
    // took the same time with and without them.
    return n < ((int64_t)1 << 31) && o.accum_mode == 0 && o.bin_mode == 0 &&
           (!L.tiles || n <= WIDE_MAX) && L.acc_form == 0 && L.block_threads == BLOCK;
}

bool fused_stores_once(int64_t n, const qdot_options &o)
{
    // k_resweep reads the result that it completes
    return !o.guard_mode || n <= ONE_BLOCK_MAX;
}

hipError_t launch_fused(const Launch &L, const double *x, const double *y, int64_t n, double tol,
                        const qdot_options &o, qdot_result *out)
{
    return launch_fused_t<double>(L, x, y, n, tol, o, out);
}

hipError_t launch_fused(const Launch &L, const float *x, const float *y, int64_t n, double tol,
                        const qdot_options &o, qdot_result *out)
{
    return launch_fused_t<float>(L, x, y, n, tol, o, out);
}

}  // namespace qd
