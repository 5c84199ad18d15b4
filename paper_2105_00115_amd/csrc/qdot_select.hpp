// The selection of one qdot by one block, from counts in its LDS, and the
// pieces around it that the kernels share: the counting of components and the
// whole result from the selection and the class sums.
#pragma once

#include "qdot_blocks.hpp"

namespace qd {

struct SelArgs {
    int key_mode, score_mode, nonstrict, mu_single;
    double tol;
};

// Counts 4 components into the LDS histogram h; sg collects bit 0 for a
// negative and bit 1 for a positive non-zero product.
template <class T>
__device__ __forceinline__ void count4(const T *xv, const T *yv, int lim, int key_mode,
                                       unsigned int *h, unsigned int &sg)
{
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const auto c = [&]() {
            if constexpr (sizeof(T) == 4) return component_f(xv[e], yv[e], key_mode);
            else return component(xv[e], yv[e], key_mode);
        }();
        const bool valid = e < lim;
        sg |= (valid & !c.zero) ? (c.sgn ? 1u : 2u) : 0u;
        // zero products land in FH_ZERO, non-finite ones in FH_BAD
        if (valid) atomicAdd(&h[c.slot + (c.bad ? 1 : 0)], 1u);
    }
}

__device__ __forceinline__ void count_signs(unsigned int sg, unsigned int *h)
{
    const bool neg = __ballot(sg & 1u) != 0ull, pos = __ballot(sg & 2u) != 0ull;
    if ((threadIdx.x & 63) == 0) {
        if (neg) atomicAdd(&h[FH_NEG], 1u);
        if (pos) atomicAdd(&h[FH_POS], 1u);
    }
}

// ---------------------------------------------------------------------------
// Selection by one block of NT threads from the merged counts, which it holds
// in LDS (h, 4 FQ words).  Its code runs once per block and cold, so it is
// kept short: rolled loops over the live slots alone, one slot per lane.
// ---------------------------------------------------------------------------
struct Sel {
    int e_max, e_min, n_bins, t, c32;
    unsigned int n_zero, signs;
    int status;  // QDOT_OK, or the error that the result reports
    int kept;    // some component is not perforated
    __device__ bool live() const { return status == QDOT_OK && n_bins > 0; }
};

template <int NT>
struct SelLds {
    int top, bot, bins;  // highest and lowest live slot, live slots
    int kept;            // some class is not perforated
    unsigned int cnt[NT / 64][3];
    double bound[CUT_THREADS / 64];
    int unatt[NT / 64];
    double sum;          // S of the combine (units of 2^e_max)
    qdot_result sums;    // value, parts and overflow flag of the combine
};

// Before find_window, with a barrier between.
template <int NT>
__device__ __forceinline__ void select_begin(SelLds<NT> &S)
{
    if (threadIdx.x == 0) {
        S.top = -1;
        S.bot = W;
        S.bins = 0;
        S.kept = 0;
    }
}

// Live slots of the calling thread's quads v (quad k NT + tid is v[k]) into
// S; a barrier has to follow.
template <int NT, int K>
__device__ __forceinline__ void find_window(const uint4 (&v)[K], SelLds<NT> &S)
{
    int top = -1, bot = W, bins = 0;
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int q = k * NT + (int)threadIdx.x;
        if (q >= FQ - 1 || !(v[k].x | v[k].y | v[k].z | v[k].w)) continue;
        top = 4 * q + (v[k].w ? 3 : v[k].z ? 2 : v[k].y ? 1 : 0);
        bot = min(bot, 4 * q + (v[k].x ? 0 : v[k].y ? 1 : v[k].z ? 2 : 3));
        bins += (v[k].x ? 1 : 0) + (v[k].y ? 1 : 0) + (v[k].z ? 1 : 0) + (v[k].w ? 1 : 0);
    }
    // few waves hold live slots
    if (__ballot(bins) != 0ull) {
        top = wave_reduce_i(top, [](int p, int r) { return max(p, r); });
        bot = wave_reduce_i(bot, [](int p, int r) { return min(p, r); });
        bins = wave_reduce_i(bins, [](int p, int r) { return p + r; });
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&S.top, top);
            atomicMin(&S.bot, bot);
            atomicAdd(&S.bins, bins);
        }
    }
}

__device__ __forceinline__ uint4 ld_dev_quad(const uint4 *p)
{
    const unsigned long long *w = reinterpret_cast<const unsigned long long *>(p);
    const unsigned long long a = ld_dev(w), b = ld_dev(w + 1);
    return make_uint4((unsigned int)a, (unsigned int)(a >> 32), (unsigned int)b,
                      (unsigned int)(b >> 32));
}

__device__ __forceinline__ int sigma_of(unsigned int m, int slot, const Sel &s)
{
    // eq. (bin-score-def) with exact bins
    const int cl = m <= 1u ? 0 : 32 - __clz((int)(m - 1u));
    return cl + slot + KMIN - s.e_max - s.t + 1;
}

__device__ __forceinline__ int sel_class(int sigma, int nonstrict, int mu_single)
{
    const int c = class_of(sigma, nonstrict);
    return mu_single && c == QDOT_DOUBLE ? SINGLE_IN : c;
}

// e_max, e_min, N_bins and t from the window in S, and the classes of the
// slots in it (perforated where empty) and of the zero slot into lut: the
// only ones that a component can have.  up: the counts are those of a sample
// of one component in 2^up.  Every thread calls it, after a barrier that
// completes h and the window; it ends with one.
template <int NT>
__device__ __forceinline__ Sel select_classes(const unsigned int *h, const SelArgs &a,
                                              SelLds<NT> &S, unsigned char *lut, int up = 0)
{
    const int tid = threadIdx.x;
    const int top = S.top, bot = S.bot;
    Sel s;
    s.n_bins = S.bins;
    s.e_max = top + KMIN;
    s.e_min = bot + KMIN;
    s.t = s.n_bins
              ? floor_log2_ratio(a.tol, a.score_mode == 0 ? (unsigned long long)s.n_bins : 1ull)
              : 0;
    s.c32 = s.e_max + s.t + 22;
    s.n_zero = h[FH_ZERO];
    const bool tol_ok = a.tol > 0.0 && !__builtin_isinf(a.tol);
    s.status = h[FH_BAD] ? QDOT_E_NONFINITE : tol_ok ? QDOT_OK : QDOT_E_INVAL;
    s.signs = (h[FH_NEG] ? 1u : 0u) | (h[FH_POS] ? 2u : 0u);
#pragma unroll 1
    for (int j = bot + tid; j <= top; j += NT) {
        const unsigned int m = h[j];
        const int cls = m ? sel_class(sigma_of(m, j, s) + up, a.nonstrict, a.mu_single)
                          : QDOT_PERF;
        lut[j] = (unsigned char)cls;
        if (cls != QDOT_PERF) S.kept = 1;
    }
    if (tid == 0) lut[ZERO_SLOT] = (unsigned char)QDOT_PERF;
    __syncthreads();
    s.kept = S.kept;
    return s;
}

// Counts per class, the bound's sums and the unattainable flag into S.  The
// bound is summed in block_cutoff's order (that of a workgroup of CUT_THREADS
// threads, one slot per thread from the lowest live one), so it is the same
// bit for bit: wave by wave of 64 slots, and the waves' sums in finish_result.
// Every thread calls it; a barrier has to follow.
template <int NT>
__device__ __forceinline__ void select_count(const unsigned int *h, const Sel &s,
                                             const SelArgs &a, SelLds<NT> &S)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int cd = 0, cs = 0, ch = 0, unatt = 0;
    const int ulim = (a.mu_single ? 23 : 52) + (a.nonstrict ? 1 : 0);
    const int bot = s.e_min - KMIN, top = s.e_max - KMIN;
#pragma unroll 1
    for (int w = wv; w < CUT_THREADS / 64; w += NT / 64) {
        double bound = 0.0;
#pragma unroll 1
        for (int j = bot + w * 64 + lane; j <= top; j += CUT_THREADS) {
            const unsigned int m = h[j];
            if (!m) continue;
            const int sigma = sigma_of(m, j, s);
            const int cls = sel_class(sigma, a.nonstrict, a.mu_single);
            unatt |= sigma >= ulim;
            cd += cls == QDOT_DOUBLE ? (int)m : 0;
            cs += (cls == QDOT_SINGLE || cls == SINGLE_IN) ? (int)m : 0;
            ch += cls == QDOT_HALF ? (int)m : 0;
            // Thm 3.3 term M_k 2^(k - e_max + 1) eps(class)
            bound += ldexp((double)m * eps_of_class(cls), j + KMIN - s.e_max + 1);
        }
        if (bot + w * 64 <= top) bound = wave_sum_d(bound);
        if (lane == 0) S.bound[w] = bound;
    }
    auto add = [](int p, int r) { return p + r; };
    cd = wave_reduce_i(cd, add);
    cs = wave_reduce_i(cs, add);
    ch = wave_reduce_i(ch, add);
    const bool ua = __ballot(unatt) != 0ull;
    if (lane == 0) {
        S.cnt[wv][0] = (unsigned int)cd;
        S.cnt[wv][1] = (unsigned int)cs;
        S.cnt[wv][2] = (unsigned int)ch;
        S.unatt[wv] = ua;
    }
}

// The result's fields that follow from the selection and select_count's sums,
// as block_cutoff forms them; value and parts are those of an empty sum.  One
// thread calls it, after a barrier.
template <int NT>
__device__ __forceinline__ void result_fields(const Sel &s, const SelArgs &a, int64_t n,
                                              const SelLds<NT> &S, qdot_result &R)
{
    constexpr int NW = NT / 64;
    long long c[3] = {0, 0, 0};
    double b = 0.0;
    int u = 0;
#pragma unroll
    for (int w = 0; w < NW; w++) {
        for (int q = 0; q < 3; q++) c[q] += S.cnt[w][q];
        u |= S.unatt[w];
    }
#pragma unroll
    for (int w = 0; w < CUT_THREADS / 64; w++) b += S.bound[w];
    const bool live = s.live(), bad = s.status != QDOT_OK;
    const bool none = c[0] + c[1] + c[2] == 0;
    int flags = u ? QDOT_F_UNATTAINABLE : 0;
    // Thm 3.6, as in block_cutoff
    if ((long long)s.e_max - s.e_min <= -(long long)s.t - (a.mu_single ? 10 : 23))
        flags |= QDOT_F_THM_ALL_DOUBLE;
    if (none) flags |= QDOT_F_ALL_PERF;
    // an error result: status and a NaN value, every other field 0
    R.status = s.status;
    R.value = bad ? __longlong_as_double(0x7ff8000000000000ll) : 0.0;
    R.part[0] = R.part[1] = R.part[2] = 0.0;
    R.n_zero = bad ? 0 : s.n_zero;
    R.n_bins = live ? s.n_bins : 0;
    R.e_max = R.e_ref = live ? s.e_max : 0;
    R.e_min = live ? s.e_min : 0;
    R.t = live ? s.t : 0;
    R.count[QDOT_DOUBLE] = live ? c[0] : 0;
    R.count[QDOT_SINGLE] = live ? c[1] : 0;
    R.count[QDOT_HALF] = live ? c[2] : 0;
    R.count[QDOT_PERF] = bad ? 0 : live ? n - c[0] - c[1] - c[2] : n;
    R.bound_rel = live ? b : 0.0;
    R.bound_abs = live ? ldexp(b, s.e_max) : 0.0;
    R.lower = 0.0;
    R.passes = live && !none ? 1 : 0;
    R.flags = bad ? 0 : live ? flags : QDOT_F_ALL_PERF;
}

// The whole result into R: wave 0 forms result_fields, wave 1 the class sums
// (red, per wave, as block_reduce3_waves leaves them) with combine_value,
// both at the same time.  e_sum, c32_sum: the units of the sums (2^e_max and
// 2^c32, or those of a guess).  Every thread calls it, after a barrier; it
// ends with one.  The sum before scaling is left in S.sum (0 when nothing was
// kept).
template <int NT>
__device__ __forceinline__ void finish_result(const Sel &s, const SelArgs &a, int64_t n,
                                              SelLds<NT> &S, Acc (*red)[NT / 64], qdot_result &R,
                                              int e_sum, int c32_sum)
{
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x;
    if (tid == 0) result_fields<NT>(s, a, n, S, R);
    if (tid >> 6 == 1) {
        // one lane per class, then the three together
        const int lane = tid & 63, q = lane < 3 ? lane : 0;
        Acc b = red[q][0];
#pragma unroll
        for (int w = 1; w < NW; w++) b = acc_merge(b, red[q][w]);
        Acc f[3];
#pragma unroll
        for (int c = 0; c < 3; c++) f[c] = Acc{__shfl(b.s, c, 64), __shfl(b.c, c, 64)};
        if (lane == 0) {
            S.sum = 0.0;
            if (s.live()) S.sum = combine_value(f, e_sum, c32_sum, 0, &S.sums, a.mu_single);
        }
    }
    __syncthreads();
    if (tid == 0 && s.live()) {
        R.value = S.sums.value;
        for (int c = 0; c < 3; c++) R.part[c] = S.sums.part[c];
        R.flags |= S.sums.flags;
    }
    __syncthreads();
}

template <int NT>
__device__ __forceinline__ void finish_result(const Sel &s, const SelArgs &a, int64_t n,
                                              SelLds<NT> &S, Acc (*red)[NT / 64], qdot_result &R)
{
    finish_result<NT>(s, a, n, S, red, R, s.e_max, s.c32);
}

// Per-wave sums of three accumulators into red (a barrier has to follow).
// The FP32 classes' accumulators are held by the first lane of each 16-lane
// row alone (acc_group), unless ALL.
template <int NT, bool ALL>
__device__ __forceinline__ void block_reduce3_waves(Acc a[3], Acc (*red)[NT / 64])
{
    a[0] = wave_reduce_rows(a[0]);
#pragma unroll
    for (int q = 1; q < 3; q++) {
        a[q] = ALL ? wave_reduce_rows(a[q]) : wave_merge_rows(a[q]);
    }
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < 3; q++) red[q][threadIdx.x >> 6] = a[q];
}

}  // namespace qd
