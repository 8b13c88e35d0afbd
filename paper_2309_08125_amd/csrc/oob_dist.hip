// Batch distribution (Section 4.2.2, Eq. 6 of the Oobleck paper) and the choice of the plan by
// throughput, for gfx950.  One lane solves one plan, exactly.
//
// Method.  For a fixed level mu,  min sum_i (N_i T_i - mu)^2  over sum N_i = Q, N_i >= 1  is a
// separable convex allocation: rounding mu / T_i and then adding or removing microbatches one at
// a time where that is cheapest gives its optimum, and as mu grows the optimum changes by single
// exchanges of one microbatch from a faster to a slower pipeline, each at a level that is a ratio
// of integers.  Every allocation on that path is feasible for Eq. 6, and at mu = the mean of an
// optimum of Eq. 6 the path holds such an optimum (the sum of squares around the mean IS the
// variance, and no allocation has a smaller one), so the smallest variance met on the path is
// the minimum.  Any feasible allocation bounds the part of the path that matters.  Let V be its
// sum of squared deviations, m an optimum's mean and d_i = N_i T_i - m: sum d_i = 0, sum d_i^2 <= V, and
// from Q = sum_i (m + d_i) / T_i with H = sum_i 1 / T_i
//     |m - Q / H| = |sum_i d_i (1 / T_i - H / x)| / H <= sqrt(V) sqrt(sum_i (1 / T_i - H / x)^2) / H
// (x pipelines; Cauchy-Schwarz): the closer the times, the shorter the path.
//
// Pipelines of one template have the same T and stay within one microbatch of each other, so the
// state of a plan is one total per template in use (at most 16), kept in LDS with one column
// per lane (192 bytes a lane; the templates' times are one table per workgroup); a template's
// donor is one of its fullest pipelines, its receiver one of its emptiest.  Products reach
// 2^124: all exact arithmetic is in 128-bit integers.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "oob_dist.h"
#include "oob_plan.h"

namespace oob_dist {

typedef __int128 i128;
constexpr int kLanes = 64; // plans per workgroup: a few thousand plans already reach every compute unit
constexpr int kLoads = 8;  // counts of a plan in flight while its templates are listed
constexpr int kT = OOB_DIST_MAX_TEMPLATES_IN_PLAN;
constexpr long long kMaxExchanges = 1ll << 24; // never reached (at most Q exchanges per template): every lane's loop ends

struct Args {
    const unsigned short *x;
    long long count, capacity;
    int p;
    const long long *tT;
    int Q;
    unsigned long long *vx;
    long long *slowest;
    unsigned short *base, *extra;
    int *status;
};

// One plan's state: column `lane` of arrays [kT][kLanes].  Template k of the plan has x pipelines;
// e of them hold n + 1 microbatches, the others n (0 <= e < x): no division in the loops.
struct Plan {
    const double *tT;              // the workgroup's copy of the templates' times per microbatch (integers: exact)
    unsigned short *j, *x, *n, *e; // template index; pipelines; see above
    int t, xs;                     // templates in use; pipelines in all
    __device__ double Td(int k) const { return tT[j[k * kLanes]]; }
    __device__ long long Tk(int k) const { return (long long)Td(k); }
    __device__ int xk(int k) const { return x[k * kLanes]; }
    __device__ int fullest(int k) const { return n[k * kLanes] + (e[k * kLanes] > 0); } // microbatches of a fullest pipeline
    __device__ int emptiest(int k) const { return n[k * kLanes]; }
    __device__ void take(int k) const { // one microbatch less for a fullest pipeline
        if (e[k * kLanes] > 0) e[k * kLanes] -= 1;
        else { n[k * kLanes] -= 1; e[k * kLanes] = (unsigned short)(xk(k) - 1); }
    }
    __device__ void give(int k) const { // one more for an emptiest pipeline
        if (e[k * kLanes] + 1 == xk(k)) { n[k * kLanes] += 1; e[k * kLanes] = 0; }
        else e[k * kLanes] += 1;
    }
};

// Comparisons of exact integers are decided in doubles where the difference exceeds the rounding of the
// double expressions, and in 128 bits otherwise (a 128-bit product is some forty instructions, a double one
// instruction; random times leave about one comparison in 10^8 to the exact form).  kEps bounds the rounding of a sum of
// two products of three factors relative to the sum of their magnitudes (five roundings of 2^-53, doubled).
constexpr double kEps = 1.0 / (1ll << 49);

// The optimum of the fixed-level problem at the integer level mu >= 0.
__device__ void allocate_at(const Plan &pl, long long mu, int Q) {
    long long tot = 0;
    for (int k = 0; k < pl.t; ++k) {
        const long long T = pl.Tk(k), num = 2 * mu + T; // num < 2^53
        long long n = (long long)((double)num / (double)(2 * T)); // nearest integer to mu / T, once corrected
        n -= n * (2 * T) > num;
        n += (n + 1) * (2 * T) <= num;
        if (n < 1) n = 1;
        if (n > Q) n = Q;
        pl.n[k * kLanes] = (unsigned short)n;
        pl.e[k * kLanes] = 0;
        tot += n * pl.xk(k);
    }
    // cost of one microbatch more or less for a pipeline of T that counts as m (odd, its sign that of the change):
    // T^2 m - 2 T mu (add, m = 2 n + 1) or T^2 m + 2 T mu (remove, m = 1 - 2 n)
    const bool remove = tot > Q;
    const double mud = remove ? 2.0 * (double)mu : -2.0 * (double)mu;
    while (tot != Q) {
        int arg = -1, am = 0;
        double bc = 0, be = 0;
        for (int k = 0; k < pl.t; ++k) {
            const int m = remove ? 1 - 2 * pl.fullest(k) : 2 * pl.emptiest(k) + 1;
            if (remove && m > -3) continue; // it holds one microbatch
            const double T = pl.Td(k), p = T * T * m, q = T * mud, c = p + q, e = (fabs(p) + fabs(q)) * kEps;
            bool less = c < bc;
            if (arg >= 0 && fabs(c - bc) <= e + be) {
                const long long Ti = (long long)T, Tb = pl.Tk(arg), s = remove ? 2 * mu : -2 * mu;
                less = (i128)Ti * Ti * m + (i128)Ti * s < (i128)Tb * Tb * am + (i128)Tb * s;
            }
            if (arg < 0 || less) { bc = c; be = e; arg = k; am = m; }
        }
        if (arg < 0) break; // cannot happen: tot > Q >= pipelines, so some pipeline holds two
        if (remove) { pl.take(arg); --tot; } else { pl.give(arg); ++tot; }
    }
}

// S1 = sum a_i, S2 = sum a_i^2 over the pipelines (a_i = N_i T_i).
__device__ void sums(const Plan &pl, i128 *S1, i128 *S2) {
    i128 s1 = 0, s2 = 0;
    for (int k = 0; k < pl.t; ++k) {
        const i128 T = pl.Tk(k);
        const int n = pl.n[k * kLanes], e = pl.e[k * kLanes]; // e pipelines hold n + 1, the others n
        const i128 lo = T * n, hi = T * (n + 1);
        s1 += lo * (pl.xk(k) - e) + hi * e;
        s2 += lo * lo * (pl.xk(k) - e) + hi * hi * e;
    }
    *S1 = s1; *S2 = s2;
}

// The level of the exchange d -> r as a fraction: c / w (see the loop below).
__device__ i128 exchange_c(const Plan &pl, int d, int r) {
    const long long Td = pl.Tk(d), Tr = pl.Tk(r);
    return (i128)Td * Td * (1 - 2 * pl.fullest(d)) + (i128)Tr * Tr * (1 + 2 * pl.emptiest(r));
}
__device__ long long exchange_w(const Plan &pl, int d, int r) { return 2 * (pl.Tk(r) - pl.Tk(d)); } // below 2^37
__device__ bool exact_less(const Plan &pl, int d, int r, int bd, int br) {
    return exchange_c(pl, d, r) * exchange_w(pl, bd, br) < exchange_c(pl, bd, br) * exchange_w(pl, d, r);
}
__device__ bool level_above(const Plan &pl, int d, int r, i128 mu) { return exchange_c(pl, d, r) > exchange_w(pl, d, r) * mu; }

// What bounds it: the vector ALUs, on chains of LDS reads at three waves per SIMD; the bytes of a plan (6 p + 28) would
// take a fifth of the time.  1 343 380 plans of up to 57 templates, 512 microbatches: 1.24 -> 0.49 ms by the shorter path,
// comparisons in doubles, counts read eight at a time and every entry of base and extra written once.
__global__ void __launch_bounds__(kLanes) k_dist_solve(Args a) {
    HIP_DYNAMIC_SHARED(double, s_tT) // [p]
    __shared__ unsigned short s_x[kT * kLanes], s_j[kT * kLanes], s_n[kT * kLanes], s_e[kT * kLanes];
    __shared__ unsigned short s_bn[kT * kLanes], s_be[kT * kLanes]; // the best allocation met so far
    const int lane = threadIdx.x;
    for (int j = lane; j < a.p; j += kLanes) s_tT[j] = (double)a.tT[j]; // exact where it is used (up to 2^35)
    __syncthreads();
    const long long i = (long long)blockIdx.x * kLanes + lane;
    if (i >= a.count) return;
    Plan pl;
    pl.tT = s_tT; pl.j = s_j + lane; pl.x = s_x + lane; pl.n = s_n + lane; pl.e = s_e + lane;
    unsigned short *bn = s_bn + lane, *be = s_be + lane, *tj = s_j + lane;

    // the templates in use
    int t = 0, xs = 0, st = OOB_DIST_OK;
    for (int j0 = 0; j0 < a.p; j0 += kLoads) {
        int c[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) c[q] = j0 + q < a.p ? a.x[(long long)(j0 + q) * a.capacity + i] : 0;
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            if (!c[q] || st != OOB_DIST_OK) continue;
            const double T = s_tT[j0 + q]; // a time beyond 2^53 is rounded, and refused all the same
            if (t == kT) { st = OOB_DIST_TOO_MANY_TEMPLATES; continue; }
            if (T < 1 || T > (double)OOB_DIST_MAX_T) { st = OOB_DIST_BAD_TIME; continue; }
            pl.x[t * kLanes] = (unsigned short)c[q]; tj[t * kLanes] = (unsigned short)(j0 + q);
            xs += c[q];
            ++t;
        }
    }
    if (st == OOB_DIST_OK && t == 0) st = OOB_DIST_NO_PIPELINE;
    if (st == OOB_DIST_OK && xs > a.Q) st = OOB_DIST_TOO_FEW_MICROBATCHES;
    a.status[i] = st;
    if (st != OOB_DIST_OK) {
        a.vx[2 * i] = 0; a.vx[2 * i + 1] = 0; a.slowest[i] = 0;
        if (a.base)
            for (int j = 0; j < a.p; ++j) {
                a.base[(long long)j * a.capacity + i] = 0;
                a.extra[(long long)j * a.capacity + i] = 0;
            }
        return;
    }
    pl.t = t; pl.xs = xs;

    // the stretch of levels that can hold the optimum's mean
    double H = 0;
    bool twins = false; // two templates of the same time
    for (int k = 0; k < t; ++k) {
        const double T = pl.Td(k);
        H += (double)pl.xk(k) / T;
        for (int l = 0; l < k; ++l) twins |= pl.Td(l) == T;
    }
    double D = 0;
    for (int k = 0; k < t; ++k) {
        const double r = 1.0 / pl.Td(k) - H / xs;
        D += r * r * pl.xk(k);
    }
    const double L0 = (double)a.Q / H;
    allocate_at(pl, (long long)(L0 + 0.5), a.Q);
    i128 S1, S2;
    sums(pl, &S1, &S2);
    const double V = (double)((i128)xs * S2 - S1 * S1) / (double)xs; // sum of squared deviations of a feasible allocation
    // With twins the distribution met first among equal ones depends on where the path starts: it starts where the
    // cruder bound, sqrt(V), puts it.
    const double narrow = twins ? 1.0 : fmin(sqrt(D) / H, 1.0);
    const double R = sqrt(V) * (narrow * (1.0 + 1e-9) + 1e-12) + L0 * 1e-9 + 2.0; // widened for the rounding of these few operations
    const long long mu_lo = L0 - R > 0 ? (long long)(L0 - R) : 0;
    const i128 mu_hi = (i128)(long long)(L0 + R) + 1;

    allocate_at(pl, mu_lo, a.Q);
    sums(pl, &S1, &S2);
    i128 best = (i128)xs * S2 - S1 * S1;
    for (int k = 0; k < t; ++k) { bn[k * kLanes] = pl.n[k * kLanes]; be[k * kLanes] = pl.e[k * kLanes]; }
    for (long long step = 0; step < kMaxExchanges; ++step) {
        // the next exchange: a microbatch of a fullest pipeline of template d (n_d of them) goes to an emptiest
        // pipeline of a slower template r (n_r): it pays from the level c / w on,
        // c = T_d^2 + T_r^2 - 2 T_d^2 n_d + 2 T_r^2 n_r,  w = 2 (T_r - T_d) > 0
        int bd = -1, br = -1;
        double bc = 0, be2 = 0, bw = 1;
        for (int d = 0; d < t; ++d) {
            const int nd = pl.fullest(d);
            if (nd < 2) continue;
            const double Td = pl.Td(d), cd = Td * Td * (1 - 2 * nd);
            for (int r = 0; r < t; ++r) {
                const double Tr = pl.Td(r);
                if (Tr <= Td) continue;
                const double cr = Tr * Tr * (1 + 2 * pl.emptiest(r)), c = cd + cr, w = 2.0 * (Tr - Td); // w exact
                const double err = (cr - cd) * kEps; // cd < 0 < cr
                const double diff = c * bw - bc * w;
                bool less = diff < 0;
                if (bd >= 0 && fabs(diff) <= 2.0 * (err * bw + be2 * w)) less = exact_less(pl, d, r, bd, br);
                if (bd < 0 || less) { bc = c; be2 = err; bw = w; bd = d; br = r; }
            }
        }
        if (bd < 0 || level_above(pl, bd, br, mu_hi)) break; // past the stretch
        const long long Td = pl.Tk(bd), Tr = pl.Tk(br);
        const int nd = pl.fullest(bd), nr = pl.emptiest(br);
        S1 += Tr - Td;
        S2 += (i128)Tr * Tr * (2 * nr + 1) - (i128)Td * Td * (2 * nd - 1);
        pl.take(bd);
        pl.give(br);
        const i128 v = (i128)xs * S2 - S1 * S1;
        if (v < best) {
            best = v;
            for (int k = 0; k < t; ++k) { bn[k * kLanes] = pl.n[k * kLanes]; be[k * kLanes] = pl.e[k * kLanes]; }
        }
    }

    long long slow = 0;
    for (int k = 0; k < t; ++k) {
        const long long time = (long long)(bn[k * kLanes] + (be[k * kLanes] > 0)) * pl.Tk(k);
        slow = time > slow ? time : slow;
    }
    if (a.base) { // every entry written once
        int k = 0, next = tj[0];
        for (int j = 0; j < a.p; ++j) {
            unsigned short n = 0, e = 0;
            if (j == next) {
                n = bn[k * kLanes]; e = be[k * kLanes];
                ++k;
                next = k < t ? tj[k * kLanes] : -1;
            }
            a.base[(long long)j * a.capacity + i] = n;
            a.extra[(long long)j * a.capacity + i] = e;
        }
    }
    a.vx[2 * i] = (unsigned long long)best;
    a.vx[2 * i + 1] = (unsigned long long)(best >> 64);
    a.slowest[i] = slow;
}

// Plan choice: the smallest `slowest` among the solved plans of a group, the first of equals.
// Workgroup (g, y) reduces every s-th stretch of kChooseThreads plans of group g, s = as many workgroups as have
// kChoosePlans plans each (lanes keep the first minimum of their strided share, waves and then the workgroup combine (value, index) pairs
// lexicographically) and merges its winner into best[group] with a compare-and-swap on the index:
// `slowest` does not change during the launch, so "is plan i better than the plan best[group]
// names now" is decided by reading both values, and the loop ends as soon as the entry names a plan
// that is at least as good.  k_dist_choose_init sets every entry to -1 ("no plan") first.
// Workgroups over stretches of the whole list, which walk the groups of their stretch one after the other: 33 us for
// 1 343 380 plans in 57 groups, 32 for 10 251 in 29, 25 for a million in 4 000 groups of one size, 760 in 4 000 groups of
// five; here 15, 7, 10 and 10 us.  64 workgroups for every group, whatever its size: 25, 6, 60 and 60 us (and 865 for
// 60 000 groups, 72 here).
constexpr int kChooseThreads = 256, kChooseLoads = 4;
// Fewer plans to a workgroup than these and what takes the time is the merging, one winner of a group after the other;
// many groups get few workgroups each, because those without plans have to be launched too.
constexpr long long kChooseMaxSlices = 64, kChoosePlans = 2048, kChooseWorkgroups = 16384;
__global__ void k_dist_choose_init(long long *best, int segments) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < segments) best[g] = -1;
}
__device__ __forceinline__ bool better(long long v, long long i, long long bv, long long bi) {
    return i >= 0 && (bi < 0 || v < bv || (v == bv && i < bi));
}
__global__ void __launch_bounds__(kChooseThreads) k_dist_choose(const long long *offsets, long long count,
                                                          const long long *slowest, const int *status,
                                                          long long *best) {
    __shared__ long long s_v[kChooseThreads / 64], s_i[kChooseThreads / 64];
    const int g = blockIdx.x;
    const long long lo = offsets[g], most = offsets[0] + count, hi = offsets[g + 1] < most ? offsets[g + 1] : most;
    const long long slices = std::min<long long>(gridDim.y, (hi - lo + kChoosePlans - 1) / kChoosePlans);
    const long long stride = slices * kChooseThreads;
    if ((long long)blockIdx.y >= slices) return; // the same for the whole workgroup (every slice has plans)
    long long bv = 0, bi = -1;
    for (long long i0 = lo + (long long)blockIdx.y * kChooseThreads + threadIdx.x; i0 < hi; i0 += stride * kChooseLoads) {
        long long v[kChooseLoads];
        int st[kChooseLoads];
#pragma unroll
        for (int q = 0; q < kChooseLoads; ++q) { // past the end: the first one again
            const long long i = i0 + q * stride < hi ? i0 + q * stride : i0;
            v[q] = slowest[i];
            st[q] = status[i];
        }
#pragma unroll
        for (int q = 0; q < kChooseLoads; ++q) // ascending: a lane keeps its first minimum
            if (i0 + q * stride < hi && st[q] == OOB_DIST_OK && (bi < 0 || v[q] < bv)) { bv = v[q]; bi = i0 + q * stride; }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        const long long ov = __shfl_down(bv, d, 64), oi = __shfl_down(bi, d, 64);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if ((threadIdx.x & 63) == 0) { s_v[threadIdx.x >> 6] = bv; s_i[threadIdx.x >> 6] = bi; }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kChooseThreads / 64; ++w)
        if (better(s_v[w], s_i[w], bv, bi)) { bv = s_v[w]; bi = s_i[w]; }
    if (bi < 0) return;
    unsigned long long *slot = (unsigned long long *)&best[g];
    long long cur = (long long)atomicAdd(slot, 0ull); // coherent read of the entry
    while (better(bv, bi, cur >= 0 ? slowest[cur] : 0, cur)) {
        const long long seen = (long long)atomicCAS(slot, (unsigned long long)cur, (unsigned long long)bi);
        if (seen == cur) break;
        cur = seen;
    }
}

} // namespace oob_dist

extern "C" int oob_dist_solve(const uint16_t *x, int64_t count, int64_t capacity, int p, const int64_t *template_T,
                              int Q, uint64_t *vx, int64_t *slowest, uint16_t *base, uint16_t *extra,
                              int32_t *status, void *stream) {
    using namespace oob_dist;
    if (!x || !template_T || !vx || !slowest || !status || (base == nullptr) != (extra == nullptr)) return OOB_EINVAL;
    if (count < 0 || capacity < count || p < 1 || p > OOB_DIST_MAX_TEMPLATES || Q < 1 || Q > OOB_DIST_MAX_Q) return OOB_EINVAL;
    if (count == 0) return OOB_OK;
    const long long blocks = (count + kLanes - 1) / kLanes;
    if (blocks > 0x7fffffffll) return OOB_EINVAL;
    Args a;
    a.x = x; a.count = count; a.capacity = capacity; a.p = p; a.tT = (const long long *)template_T; a.Q = Q;
    a.vx = (unsigned long long *)vx; a.slowest = (long long *)slowest; a.base = base; a.extra = extra; a.status = status;
    hipLaunchKernelGGL(k_dist_solve, dim3((unsigned)blocks), dim3(kLanes), (size_t)p * sizeof(double), (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? OOB_OK : OOB_EHIP;
}

extern "C" int oob_dist_choose(const int64_t *offsets, int segments, int64_t count, const int64_t *slowest,
                               const int32_t *status, int64_t *best, void *stream) {
    using namespace oob_dist;
    if (!offsets || !slowest || !status || !best || segments < 0 || count < 0) return OOB_EINVAL;
    if (segments == 0) return OOB_OK;
    const long long slices = std::min({(count + kChoosePlans - 1) / kChoosePlans, kChooseMaxSlices,
                                       std::max(1ll, kChooseWorkgroups / segments)});
    hipLaunchKernelGGL(k_dist_choose_init, dim3((unsigned)((segments + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       (long long *)best, segments);
    if (slices > 0)
        hipLaunchKernelGGL(k_dist_choose, dim3((unsigned)segments, (unsigned)slices), dim3(kChooseThreads), 0, (hipStream_t)stream,
                           (const long long *)offsets, (long long)count, (const long long *)slowest, status, (long long *)best);
    return hipGetLastError() == hipSuccess ? OOB_OK : OOB_EHIP;
}
