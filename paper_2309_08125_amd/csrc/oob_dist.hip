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
// state of a plan is one total per template in use (at most 16); a template's
// donor is one of its fullest pipelines, its receiver one of its emptiest.  Products reach
// 2^124: all exact arithmetic is in 128-bit integers.
//
// Three forms of the same solution.  Of the plans of a node specification one in sixty has an exchange on its path at all: whether
// there is one is decided from the templates one by one (solve_in_registers), and the others are done after one allocation.  The
// few with a path wait until a wave is full of them; solve_general, in LDS and slow, keeps the plans of more than kFast
// templates and the comparisons that doubles leave open.
//
// What bounds it: the vector ALUs (3 300 instructions a wave for 57 templates, two fifths of them for reading the counts and writing the
// distribution) and, for plans with a path, waves of a few lanes that wait for memory.  1 343 380 plans of up to 57 templates, 512
// microbatches: 521 us with solve_general for every plan, 172 us for the first launch and 85 us for the second here (the walkers followed
// at the end of each wave's share 350 us; with all 57 counts of a walker read once more, and written, 172 and 170 us); 10 251 plans of
// 29 templates 41 -> 27 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "oob_dist.h"
#include "oob_plan.h"

namespace oob_dist {

typedef __int128 i128;
constexpr int kLanes = 64;  // plans side by side in a wave
constexpr int kLoads = 16;  // counts of a plan in flight while its templates are listed
constexpr int kT = OOB_DIST_MAX_TEMPLATES_IN_PLAN;
constexpr int kGeneral = 32; // lanes of a wave that solve_general uses: half of them leave room in LDS for more waves
constexpr int kFirstThreads = 256;
// Plans that a wave of the second launch looks through: some sixteen of them have a path.  512, 1 024, 2 048: 288, 283, 316 us
// for the whole call with the choice (1 343 380 plans).
constexpr int kSpanBits = 10, kSpan = 1 << kSpanBits;
// Plans up to which one launch does it all, each wave 64 plans with their paths: as many as the GPU holds at once.  What counts
// there is how long one wave takes (10 251 plans: 27 us, 15 + 33 us in two launches).
constexpr long long kOnce = 3072 * 64;
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
    int lists; // base and extra may hold what the first launch leaves to the second
};

// One plan's state: column `lane` of arrays [kT][kGeneral].  Template k of the plan has x pipelines;
// e of them hold n + 1 microbatches, the others n (0 <= e < x): no division in the loops.
struct Plan {
    const double *tT;              // the workgroup's copy of the templates' times per microbatch (integers: exact)
    unsigned short *j, *x, *n, *e; // template index; pipelines; see above
    int t, xs;                     // templates in use; pipelines in all
    __device__ double Td(int k) const { return tT[j[k * kGeneral]]; }
    __device__ long long Tk(int k) const { return (long long)Td(k); }
    __device__ int xk(int k) const { return x[k * kGeneral]; }
    __device__ int fullest(int k) const { return n[k * kGeneral] + (e[k * kGeneral] > 0); } // microbatches of a fullest pipeline
    __device__ int emptiest(int k) const { return n[k * kGeneral]; }
    __device__ void take(int k) const { // one microbatch less for a fullest pipeline
        if (e[k * kGeneral] > 0) e[k * kGeneral] -= 1;
        else { n[k * kGeneral] -= 1; e[k * kGeneral] = (unsigned short)(xk(k) - 1); }
    }
    __device__ void give(int k) const { // one more for an emptiest pipeline
        if (e[k * kGeneral] + 1 == xk(k)) { n[k * kGeneral] += 1; e[k * kGeneral] = 0; }
        else e[k * kGeneral] += 1;
    }
};

// Comparisons of exact integers are decided in doubles where the difference exceeds the rounding of the
// double expressions, and in 128 bits otherwise (a 128-bit product is some forty instructions, a double one
// instruction; random times leave about one comparison in 10^8 to the exact form).  kEps bounds the rounding of a sum of
// two products of three factors relative to the sum of their magnitudes (five roundings of 2^-53, doubled).
constexpr double kEps = 1.0 / (1ll << 49);
constexpr double kHuge = __builtin_huge_val();

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
        pl.n[k * kGeneral] = (unsigned short)n;
        pl.e[k * kGeneral] = 0;
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
        const int n = pl.n[k * kGeneral], e = pl.e[k * kGeneral]; // e pipelines hold n + 1, the others n
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

// The arrays of one wave's plans in LDS.
struct General {
    unsigned short x[kT * kGeneral], j[kT * kGeneral], n[kT * kGeneral], e[kT * kGeneral];
    unsigned short bn[kT * kGeneral], be[kT * kGeneral]; // the best allocation met so far
};

// Plan i by one lane, whatever its templates and its path.
__device__ void solve_general(const Args &a, const double *s_tT, General &g, long long i, int lane) {
    Plan pl;
    pl.tT = s_tT; pl.j = g.j + lane; pl.x = g.x + lane; pl.n = g.n + lane; pl.e = g.e + lane;
    unsigned short *bn = g.bn + lane, *be = g.be + lane, *tj = g.j + lane;

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
            pl.x[t * kGeneral] = (unsigned short)c[q]; tj[t * kGeneral] = (unsigned short)(j0 + q);
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
    for (int k = 0; k < t; ++k) { bn[k * kGeneral] = pl.n[k * kGeneral]; be[k * kGeneral] = pl.e[k * kGeneral]; }
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
            for (int k = 0; k < t; ++k) { bn[k * kGeneral] = pl.n[k * kGeneral]; be[k * kGeneral] = pl.e[k * kGeneral]; }
        }
    }

    long long slow = 0;
    for (int k = 0; k < t; ++k) {
        const long long time = (long long)(bn[k * kGeneral] + (be[k * kGeneral] > 0)) * pl.Tk(k);
        slow = time > slow ? time : slow;
    }
    if (a.base) { // every entry written once
        int k = 0, next = tj[0];
        for (int j = 0; j < a.p; ++j) {
            unsigned short n = 0, e = 0;
            if (j == next) {
                n = bn[k * kGeneral]; e = be[k * kGeneral];
                ++k;
                next = k < t ? tj[k * kGeneral] : -1;
            }
            a.base[(long long)j * a.capacity + i] = n;
            a.extra[(long long)j * a.capacity + i] = e;
        }
    }
    a.vx[2 * i] = (unsigned long long)best;
    a.vx[2 * i + 1] = (unsigned long long)(best >> 64);
    a.slowest[i] = slow;
}

// Plan i by one lane with its templates in registers: the same method and the same order of comparisons as
// solve_general, for plans of at most kFast templates.  kHard: a plan of more, one that cannot be solved, or a comparison
// that needs the exact form; solve_general takes it.
//
// Mostly no exchange lies on the stretch, and then nothing has to be searched.  A distribution is the only optimum at a level mu if every
// exchange of a microbatch between two templates costs: taking one from a fullest pipeline of d adds A = T_d^2 (1 - 2 n_d) + 2
// T_d mu, giving it to an emptiest one of r B = T_r^2 (1 + 2 n_r) - 2 T_r mu, and A + B > 0 for all d != r (the problem is
// separable and convex: a strict minimum among its neighbours is the minimum).  Where that holds for the distribution of the
// stretch's middle at both ends of the stretch, the path starts with it and has no exchange on the stretch (A + B <= 0 is what makes
// one pay).  Otherwise the path is followed with FOLLOW = true; FOLLOW = false returns kLeft.
constexpr int kFast = 10;
constexpr int kDone = 0, kLeft = 1, kHard = 2;
struct Listed { unsigned jx[kFast * kLanes], best[kFast * kLanes]; }; // template | pipelines << 16; n | e << 16 (as in Plan)
struct Walked { Listed ls; unsigned ne[kFast * kLanes]; };

// FOLLOW = false hands the list of the plan's templates over where the plan stays open: rows 0 .. t-1 of its column of base and extra hold
// them, *listed becomes t.  FOLLOW = true takes it from there if *listed is not 0.
template <bool FOLLOW> __device__ int solve_in_registers(const Args &a, const double *s_tT, Listed &ls, unsigned *ne, long long i, int lane, int *listed) {
    unsigned *const jx = ls.jx + lane, *const best_ne = ls.best + lane;
    int t = 0, xs = 0;
    if (FOLLOW && *listed) {
        t = *listed;
        unsigned w[kFast];
#pragma unroll
        for (int k = 0; k < kFast; ++k) w[k] = k < t ? (unsigned)a.base[k * a.capacity + i] | (unsigned)a.extra[k * a.capacity + i] << 16 : 0;
#pragma unroll
        for (int k = 0; k < kFast; ++k) {
            jx[k * kLanes] = w[k];
            xs += (int)(w[k] >> 16);
        }
    } else {
        for (int j0 = 0; j0 < a.p; j0 += kLoads) {
            int c[kLoads];
#pragma unroll
            for (int q = 0; q < kLoads; ++q) c[q] = j0 + q < a.p ? a.x[(long long)(j0 + q) * a.capacity + i] : 0;
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                if (!c[q]) continue;
                if (t < kFast) jx[t * kLanes] = (unsigned)(j0 + q) | (unsigned)c[q] << 16;
                xs += c[q];
                ++t;
            }
        }
        if (t == 0 || t > kFast || xs > a.Q) return kHard;
    }
    double T[kFast];
    int x[kFast], n[kFast], e[kFast];
    auto inverse = [&](int k) { return s_tT[a.p + (jx[k * kLanes] & 0xffff)]; }; // read again where it is used: registers decide how
                                                                                 // many waves run
    bool ok = true, twins = false;
    double H = 0;
#pragma unroll
    for (int k = 0; k < kFast; ++k) {
        T[k] = 1; x[k] = n[k] = e[k] = 0;
        if (k < t) {
            const unsigned w = jx[k * kLanes];
            T[k] = s_tT[w & 0xffff]; x[k] = (int)(w >> 16);
            ok &= T[k] >= 1 && T[k] <= (double)OOB_DIST_MAX_T;
            H += (double)x[k] * inverse(k);
#pragma unroll
            for (int l = 0; l < k; ++l) twins |= T[l] == T[k];
        }
    }
    if (!ok) return kHard;
    const double mean = H / xs, L0 = (double)a.Q / H;
    double D = 0;
#pragma unroll
    for (int k = 0; k < kFast; ++k)
        if (k < t) {
            const double r = inverse(k) - mean;
            D += r * r * x[k];
        }

    // every exchange costs at level mu (see above)
    auto settled = [&](double mu) {
        const double m2 = 2.0 * mu;
        double a1 = kHuge, a2 = kHuge, b1 = kHuge, b2 = kHuge; // smallest and second smallest A and B, less their rounding
        int ai = -1, bi = -1;
#pragma unroll
        for (int k = 0; k < kFast; ++k)
            if (k < t) {
                const int full = n[k] + (e[k] > 0);
                const double sq = T[k] * T[k], q = T[k] * m2, pa = sq * (2 * full - 1), pb = sq * (2 * n[k] + 1);
                const double A = full < 2 ? kHuge : (q - pa) - (q + pa) * kEps, B = (pb - q) - (pb + q) * kEps;
                a2 = fmin(a2, fmax(a1, A));
                ai = A < a1 ? k : ai;
                a1 = fmin(a1, A);
                b2 = fmin(b2, fmax(b1, B));
                bi = B < b1 ? k : bi;
                b1 = fmin(b1, B);
            }
        return (ai != bi ? a1 + b1 : fmin(a1 + b2, a2 + b1)) > 0.0;
    };
    long long mu = (long long)(L0 + 0.5), mu_hi = 0;
    long long S1; // below 2^51
    i128 S2, best;
    bool walk = false, open = false;
    for (;;) { // at the middle of the stretch, then (walk) at its lower end
#pragma unroll
        for (int k = 0; k < kFast; ++k) asm volatile("" : "+v"(T[k])); // products of the times are formed here, not kept for the next round
        // allocate_at
        const double m2 = 2.0 * (double)mu;
        int tot = 0;
#pragma unroll
        for (int k = 0; k < kFast; ++k)
            if (k < t) {
                const double num = m2 + T[k], two = 2.0 * T[k]; // integers below 2^53
                double f = floor(num * (0.5 * inverse(k))); // nearest integer to mu / T, once corrected
                f -= f * two > num ? 1.0 : 0.0;
                f += (f + 1.0) * two <= num ? 1.0 : 0.0;
                n[k] = (int)fmin(fmax(f, 1.0), (double)a.Q);
                e[k] = 0;
                tot += n[k] * x[k]; // mu is about Q / H at most, so n is at most Q / x + 2
            }
        if (tot != a.Q) {
            const bool remove = tot > a.Q;
            double c[kFast], most = 0; // what one microbatch less or more costs a template; what their rounding can come to
#pragma unroll
            for (int k = 0; k < kFast; ++k) {
                c[k] = kHuge;
                if (k < t) {
                    const double sq = T[k] * T[k], q = T[k] * m2;
                    if (remove) { if (n[k] >= 2) c[k] = q - sq * (2 * n[k] - 1); }
                    else c[k] = sq * (2 * n[k] + 1) - q;
                    most = fmax(most, 4.0 * kEps * (q + sq * (2 * n[k] + 1)));
                }
            }
            for (;;) {
                double c1 = kHuge, c2 = kHuge;
#pragma unroll
                for (int k = 0; k < kFast; ++k) {
                    c2 = fmin(c2, fmax(c1, c[k]));
                    c1 = fmin(c1, c[k]);
                }
                if (c1 >= kHuge || c2 - c1 <= most) return kHard; // (c1 is a cost: tot > Q >= pipelines, so some pipeline holds two)
#pragma unroll
                for (int k = 0; k < kFast; ++k) {
                    if (c[k] != c1) continue;
                    bool next; // the template's next pipeline starts over: another cost
                    if (remove) { // Plan::take
                        next = e[k] == 1 || x[k] == 1;
                        if (e[k] > 0) --e[k];
                        else { --n[k]; e[k] = x[k] - 1; }
                    } else {      // Plan::give
                        next = e[k] + 1 == x[k];
                        if (next) { ++n[k]; e[k] = 0; }
                        else ++e[k];
                    }
                    if (next) { // formed anew: a sum of steps would add up their roundings, which `most` does not cover
                        double Tk = T[k];
                        asm volatile("" : "+v"(Tk));
                        const double sq = Tk * Tk, q = Tk * (2.0 * (double)mu);
                        c[k] = !remove ? sq * (2 * n[k] + 1) - q : n[k] < 2 ? kHuge : q - sq * (2 * n[k] - 1);
                        most = fmax(most, 4.0 * kEps * (q + sq * (2 * n[k] + 1)));
                    }
                }
                tot += remove ? -1 : 1;
                if (tot == a.Q) break;
            }
        }
        S1 = 0; S2 = 0;
#pragma unroll
        for (int k = 0; k < kFast; ++k)
            if (k < t) {
                const long long Tk = (long long)T[k];
                const unsigned long long lo = (unsigned long long)n[k] * n[k], hi = (unsigned long long)(n[k] + 1) * (n[k] + 1);
                S1 += Tk * ((long long)n[k] * x[k] + e[k]);
                S2 += (i128)Tk * Tk * (long long)(lo * (x[k] - e[k]) + hi * e[k]);
            }
        best = (i128)xs * S2 - (i128)S1 * S1;
        if (walk) break;
        const double V = (double)best / (double)xs; // sum of squared deviations of a feasible allocation
        const double narrow = twins ? 1.0 : fmin(sqrt(D) / H, 1.0);
        const double R = sqrt(V) * (narrow * (1.0 + 1e-9) + 1e-12) + L0 * 1e-9 + 2.0;
        mu = L0 - R > 0 ? (long long)(L0 - R) : 0;
        mu_hi = (long long)(L0 + R) + 1;
        bool only = true; // one end after the other: together they take more registers than the kernel has
#pragma unroll 1
        for (int side = 0; side < 2; ++side) only &= settled(side ? (double)mu_hi : (double)mu);
        if (only) break;
        if (!FOLLOW) { open = true; break; }
        walk = true;
    }
#pragma unroll
    for (int k = 0; k < kFast; ++k)
        if (k < t) best_ne[k * kLanes] = (unsigned)n[k] | (unsigned)e[k] << 16;
    if constexpr (FOLLOW) {
        ne += lane; // the allocation once more in LDS, for the templates that give
#pragma unroll
        for (int k = 0; k < kFast; ++k)
            if (walk && k < t) ne[k * kLanes] = (unsigned)n[k] | (unsigned)e[k] << 16;
        while (walk && !settled((double)mu_hi)) {
            int bd = -1, br = -1; // the next exchange, see solve_general
            double bc = 0, be = 0, bw = 1;
            for (int d = 0; d < t; ++d) {
                const unsigned wd = ne[d * kLanes];
                const int nd = (int)(wd & 0xffff) + (wd >> 16 ? 1 : 0);
                const double Td = s_tT[jx[d * kLanes] & 0xffff], cd = Td * Td * (1 - 2 * nd);
                if (nd < 2) continue;
#pragma unroll
                for (int r = 0; r < kFast; ++r) {
                    const double Tr = T[r];
                    if (r >= t || Tr <= Td) continue;
                    const double cr = Tr * Tr * (1 + 2 * n[r]), c = cd + cr, w = 2.0 * (Tr - Td); // w exact
                    const double err = (cr - cd) * kEps, diff = c * bw - bc * w;
                    ok &= bd < 0 || fabs(diff) > 2.0 * (err * bw + be * w);
                    if (bd < 0 || diff < 0) { bc = c; be = err; bw = w; bd = d; br = r; }
                }
            }
            if (!ok) return kHard;
            if (bd < 0) break;
            const unsigned xd = jx[bd * kLanes], xr = jx[br * kLanes];
            const long long Td = (long long)s_tT[xd & 0xffff], Tr = (long long)s_tT[xr & 0xffff];
            unsigned wd = ne[bd * kLanes], wr = ne[br * kLanes];
            const int nd = (int)(wd & 0xffff) + (wd >> 16 ? 1 : 0), nr = (int)(wr & 0xffff);
            const i128 change = (i128)Tr * Tr * (2 * nr + 1) - (i128)Td * Td * (2 * nd - 1);
            if (change > (i128)(2 * (Tr - Td)) * mu_hi) break; // past the stretch
            S1 += Tr - Td;
            S2 += change;
            wd = wd >> 16 ? wd - 0x10000u : (wd - 1) | ((xd >> 16) - 1) << 16;   // Plan::take
            wr = (wr >> 16) + 1 == xr >> 16 ? (wr & 0xffff) + 1 : wr + 0x10000u; // Plan::give
            ne[bd * kLanes] = wd;
            ne[br * kLanes] = wr;
#pragma unroll
            for (int k = 0; k < kFast; ++k) {
                if (k == bd) { n[k] = (int)(wd & 0xffff); e[k] = (int)(wd >> 16); }
                if (k == br) { n[k] = (int)(wr & 0xffff); e[k] = (int)(wr >> 16); }
            }
            const i128 v = (i128)xs * S2 - (i128)S1 * S1;
            if (v < best) {
                best = v;
                for (int k = 0; k < t; ++k) best_ne[k * kLanes] = ne[k * kLanes];
            }
        }
    }
    long long slow = 0;
    for (int k = 0; k < t; ++k) {
        const unsigned w = best_ne[k * kLanes];
        const long long time = (long long)((w & 0xffff) + (w >> 16 ? 1 : 0)) * (long long)s_tT[jx[k * kLanes] & 0xffff];
        slow = time > slow ? time : slow;
    }
    if (FOLLOW && *listed) { // the other entries are zeros
        for (int k = 0; k < t; ++k) a.base[k * a.capacity + i] = a.extra[k * a.capacity + i] = 0;
        for (int k = 0; k < t; ++k) {
            const unsigned w = best_ne[k * kLanes];
            const long long at = (long long)(jx[k * kLanes] & 0xffff) * a.capacity + i;
            a.base[at] = (unsigned short)w;
            a.extra[at] = (unsigned short)(w >> 16);
        }
    } else if (a.base) { // every entry written once
        int k = 0;
        unsigned next = open ? 0 : jx[0] & 0xffff, have = open ? jx[0] : best_ne[0];
        for (int j = 0; j < a.p; ++j) {
            unsigned w = 0;
            if ((unsigned)j == next) {
                w = have;
                ++k;
                const unsigned row = k < t ? jx[k * kLanes] : 0xffffu;
                next = open && k < t ? (unsigned)k : row & 0xffff;
                have = open ? row : k < t ? best_ne[k * kLanes] : 0;
            }
            a.base[(long long)j * a.capacity + i] = (unsigned short)w;
            a.extra[(long long)j * a.capacity + i] = (unsigned short)(w >> 16);
        }
    }
    if (!FOLLOW && open) {
        *listed = t;
        return kLeft;
    }
    a.status[i] = OOB_DIST_OK;
    a.vx[2 * i] = (unsigned long long)best;
    a.vx[2 * i + 1] = (unsigned long long)(best >> 64);
    a.slowest[i] = slow;
    return kDone;
}

__device__ __forceinline__ void load_times(const Args &a, double *s_tT) { // [p], then [p] reciprocals
    for (int j = threadIdx.x; j < a.p; j += blockDim.x) {
        const double T = (double)a.tT[j]; // exact where it is used (up to 2^35)
        s_tT[j] = T;
        s_tT[a.p + j] = 1.0 / T;
    }
    __syncthreads();
}

// The plans without an exchange on their stretch; the others are marked in `status`.
constexpr int kMarked = 1 << 30; // and the templates that are listed (0: none)
__global__ void __launch_bounds__(kFirstThreads, 4) k_dist_first(Args a) {
    HIP_DYNAMIC_SHARED(double, s_tT)
    __shared__ Listed s_listed[kFirstThreads / kLanes];
    load_times(a, s_tT);
    const long long i = (long long)blockIdx.x * kFirstThreads + threadIdx.x;
    if (i >= a.count) return;
    int listed = 0;
    if (solve_in_registers<false>(a, s_tT, s_listed[threadIdx.x / kLanes], nullptr, i, threadIdx.x & (kLanes - 1), &listed) != kDone)
        a.status[i] = kMarked + listed;
}

// The marked ones of `span` consecutive plans (all of them if marked = 0), side by side: those whose path can be followed in LDS, then
// the hard ones.
__global__ void __launch_bounds__(kLanes, 3) k_dist_rest(Args a, int span, int marked) {
    HIP_DYNAMIC_SHARED(double, s_tT) // the times, then twice [span] 16-bit numbers of plans
    __shared__ union { General general; Walked walked; } s;
    unsigned short *const left = (unsigned short *)(s_tT + 2 * a.p), *const hard = left + span;
    const int lane = threadIdx.x;
    load_times(a, s_tT);
    const long long i0 = (long long)blockIdx.x * span;
    const unsigned long long below = (1ull << lane) - 1;
    int nleft = 0, nhard = 0;
    for (int o0 = 0; o0 < span; o0 += kLanes * kLoads) {
        int st[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const long long i = i0 + o0 + q * kLanes + lane;
            st[q] = o0 + q * kLanes < span && i < a.count ? marked ? a.status[i] : kMarked : 0;
        }
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const unsigned long long m = __ballot(st[q] >= kMarked);
            if (st[q] >= kMarked) left[nleft + __popcll(m & below)] = (unsigned short)((o0 + q * kLanes + lane) | (st[q] - kMarked) << kSpanBits);
            nleft += __popcll(m);
        }
    }
    __syncthreads();
    for (int q = lane; q - lane < nleft; q += kLanes) {
        const int w = q < nleft ? left[q] : 0, o = w & ((1 << kSpanBits) - 1);
        int got = kDone, listed = a.base ? w >> kSpanBits : 0;
        if (q < nleft) got = a.lists ? solve_in_registers<true>(a, s_tT, s.walked.ls, s.walked.ne, i0 + o, lane, &listed) : kHard;
        const unsigned long long m = __ballot(got == kHard);
        if (got == kHard) hard[nhard + __popcll(m & below)] = (unsigned short)o;
        nhard += __popcll(m);
    }
    __syncthreads();
    if (lane < kGeneral)
        for (int q = lane; q < nhard; q += kGeneral) solve_general(a, s_tT, s.general, i0 + hard[q], lane);
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

// Whether two arrays [p][capacity] share no entry.
static bool apart(const unsigned short *a, const unsigned short *b, int p, long long capacity) {
    const uintptr_t bytes = (uintptr_t)p * (uintptr_t)capacity * sizeof(unsigned short), u = (uintptr_t)a, v = (uintptr_t)b;
    return u < v ? v - u >= bytes : u - v >= bytes;
}

} // namespace oob_dist

extern "C" int oob_dist_solve(const uint16_t *x, int64_t count, int64_t capacity, int p, const int64_t *template_T,
                              int Q, uint64_t *vx, int64_t *slowest, uint16_t *base, uint16_t *extra,
                              int32_t *status, void *stream) {
    using namespace oob_dist;
    if (!x || !template_T || !vx || !slowest || !status || (base == nullptr) != (extra == nullptr)) return OOB_EINVAL;
    if (count < 0 || capacity < count || p < 1 || p > OOB_DIST_MAX_TEMPLATES || Q < 1 || Q > OOB_DIST_MAX_Q) return OOB_EINVAL;
    if (count == 0) return OOB_OK;
    if ((count + kLanes - 1) / kLanes > 0x7fffffffll) return OOB_EINVAL;
    Args a;
    a.x = x; a.count = count; a.capacity = capacity; a.p = p; a.tT = (const long long *)template_T; a.Q = Q;
    a.vx = (unsigned long long *)vx; a.slowest = (long long *)slowest; a.base = base; a.extra = extra; a.status = status;
    // What is left by the first launch has its list where its distribution goes, and its counts are read again if it turns out to be hard.
    // solve_general reads all counts of a plan before it writes: it takes arrays that share entries, whole rows apart.
    a.lists = !base || (apart(x, base, p, capacity) && apart(x, extra, p, capacity) && apart(base, extra, p, capacity));
    const bool twice = count > kOnce && a.lists;
    const int span = twice ? kSpan : kLanes;
    const size_t times = 2 * (size_t)p * sizeof(double);
    if (twice) hipLaunchKernelGGL(k_dist_first, dim3((unsigned)((count + kFirstThreads - 1) / kFirstThreads)), dim3(kFirstThreads), times, (hipStream_t)stream, a);
    hipLaunchKernelGGL(k_dist_rest, dim3((unsigned)((count + span - 1) / span)), dim3(kLanes), times + 2 * span * sizeof(unsigned short), (hipStream_t)stream, a, span,
                       (int)twice);
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
