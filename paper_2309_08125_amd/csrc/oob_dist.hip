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
// How far a plan's path has to be followed depends on the templates' times.  With times that grow by a factor of two over 57 sizes one plan in
// fifty has an exchange on its path at all, with times that fall as 1 / nodes a quarter to 40 %, and with times on a coarse grid most have,
// and many exact ties.  So the launches share out work by the plans that have a path, wherever they are: with many plans a first launch
// decides from the templates one by one whether there is an exchange (solve<FOLLOW = false>), finishes the others and leaves a mark, and a second
// one takes the marked plans 64 side by side.
//
// What bounds it: the vector ALUs (2 650 instructions a wave for 57 templates in the first launch, 90 us of its 150 for 1 343 380 plans), next to
// them the memory (92 us for the same loads and stores alone) and, where few plans have a path, the chain of its longest one.  Plans of up to 57 templates, 512
// microbatches, us a call: every plan by one lane in LDS at its place; with its path followed in stretches of 1 024 plans by one wave
// each, ties of two costs by the form in LDS; by marks, with the counts and the distribution two bytes a lane, sums in 128-bit integers and
// microbatches moved one by one; here:
//     1 343 380 plans, times that grow      521     261    221    200
//                      that fall as 1 / n   506   1 115    433    409
//                      all equal            837   4 317    514    368
//       200 000 plans, times that grow      147      84     70     62
//                      all equal            260   4 128    114     84
//        10 251 plans, times that grow       41      27     30     27
//                      all equal                             40     25
//       300 000 plans of 1 000 templates                  1 214    672
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "oob_dist.h"
#include "oob_plan.h"

namespace oob_dist {

typedef __int128 i128;
constexpr int kLanes = 64; // plans side by side in a wave
constexpr int kLoads = 16; // counts of a plan in flight while its templates are listed
constexpr int kT = OOB_DIST_MAX_TEMPLATES_IN_PLAN;
constexpr int kFew = 10;   // templates that have registers in the first launch at four waves a SIMD
constexpr int kFirstThreads = 256;
constexpr int kScan = 4, kSpanBits = 10; // marks in flight of a wave of the second launch; plans whose marks it looks through, at most
// Up to kOnce plans one launch does it all, two waves a SIMD: what counts there is how long the wave with the longest path takes, and
// kOnce is what the GPU holds at once (120 000 plans 54 us, in two launches 75; three waves a SIMD, which spill, 57; all three before the counts went
// through memory four rows at a time, now 44).  Up to kFollow plans the
// first launch, at three waves a SIMD, follows the paths as well, as many as the GPU holds, and leaves the plans of many templates (160 000
// plans 65 us, with the paths in the second launch 76; 200 000 plans 92 and 81; now 150 000 plans 48 and 200 000 plans 62).
constexpr long long kOnce = 2048 * 64, kFollow = 3072 * 64;
// Waves of the second launch, at most a wave for every 64 plans.  3 072, 5 120, 7 168, 10 240, for 1 343 380 plans: times that grow 239, 234, 232, 233
// us, times that fall as 1 / nodes 655, 549, 473, 434 us: the waves without a marked plan end while the others work.
constexpr int kRestWaves = 10240;
constexpr double kHuge = __builtin_huge_val();

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

// Comparisons of exact integers are decided in doubles where the difference exceeds the rounding of the
// double expressions, and in 128 bits otherwise (random times leave about one comparison in 10^8 to the exact form, times on a coarse
// grid a good part).  kEps bounds the rounding of a sum of two products of three factors relative to the sum of their magnitudes (five
// roundings of 2^-53, doubled).  Times below kExactT need no exact form: |c| < 2^40, w < 2^12 and all sums of two products are integers
// below 2^53 (times of 1 to 20, 1 343 380 plans: 5 170 -> 2 850 us).
constexpr double kEps = 1.0 / (1ll << 49);
constexpr double kExactT = 2048;

// The templates in use of plan i: jx[k * kLanes] = template | pipelines << 16, the first `rows` of them.  Returns their number.
__device__ __forceinline__ int list_templates(const Args &a, long long i, unsigned *jx, int rows, int *pipelines) {
    int t = 0, xs = 0;
    for (int j0 = 0; j0 < a.p; j0 += kLoads) {
        int c[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) c[q] = j0 + q < a.p ? a.x[(long long)(j0 + q) * a.capacity + i] : 0;
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            if (!c[q]) continue;
            if (t < rows) jx[t * kLanes] = (unsigned)(j0 + q) | (unsigned)c[q] << 16;
            xs += c[q];
            ++t;
        }
    }
    *pipelines = xs;
    return t;
}

// A wave's 64 plans i0 .. i0 + 63, all of them below `count`, go through memory together: lane 16 r + g has the plans 4 g .. 4 g + 3 of the
// rows j = r modulo 4, so one load or store of eight bytes a lane moves four whole rows of the wave (the element's alignment, two bytes, is all that
// is asked of the arrays), and `area`, kRows rows of 64 words of the wave, turns them into a plan to a lane and back.  A row at a time, a lane its
// plan's two bytes, is twelve instructions a row for the counts and eighteen for the distribution, here four and seven; 1 343 380 plans of 57
// templates take 12 us less.  The same loads and stores without the plans' solution take 92 us there; stores that pass by the caches
// (non-temporal) cost 65 us more, since a wave's part of a row is one line of 128 bytes.
typedef unsigned short u16x4 __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2), may_alias));
typedef unsigned u32x4 __attribute__((ext_vector_type(4), may_alias));
constexpr int kRows = 8, kLoad = 16, kStage = 8; // loads in flight; of them in `area` at a time, 4 kStage rows of 16-bit counts: 2 kRows of words

// What the lanes of a wave have put into LDS so far is there for all of them.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// As list_templates, for a wave; row kT of jx is overwritten.
__device__ __forceinline__ int list_wave(const Args &a, long long i0, unsigned *jx, unsigned *area, int *pipelines) {
    const int lane = threadIdx.x & (kLanes - 1), r = lane >> 4;
    const unsigned short *from = a.x + r * a.capacity + i0 + 4 * (lane & 15);
    int t = 0, xs = 0;
    for (int j0 = 0; j0 < a.p; j0 += 4 * kLoad) {
        u16x4 c[kLoad];
#pragma unroll
        for (int q = 0; q < kLoad; ++q) {
            c[q] = (u16x4)0;
            if (j0 + 4 * q + r < a.p) c[q] = *(const u16x4 *)(from + (j0 + 4 * q) * a.capacity);
        }
#pragma unroll
        for (int s = 0; s < kLoad; s += kStage) {
            unsigned long long any[kStage]; // 16 bits a row: who has plans with the template
#pragma unroll
            for (int q = 0; q < kStage; ++q) {
                const u32x2 w = __builtin_bit_cast(u32x2, c[s + q]);
                ((u32x2 *)area)[q * kLanes + lane] = w;
                any[q] = __ballot((w.x | w.y) != 0);
            }
            wave_sync();
#pragma unroll
            for (int q = 0; q < kStage; ++q)
#pragma unroll
                for (int row = 0; row < 4; ++row) {
                    if (!(any[q] >> 16 * row & 0xffff)) continue; // uniform
                    const unsigned n = ((const unsigned short *)area)[(4 * q + row) * kLanes + lane];
                    jx[std::min(t, kT) * kLanes] = (unsigned)(j0 + 4 * (s + q) + row) | n << 16; // overwritten by the next one if there are none
                    xs += (int)n;
                    t += n != 0;
                }
            wave_sync();
        }
    }
    *pipelines = xs;
    return t;
}

// A time beyond 2^53 is rounded, and refused all the same.
__device__ __forceinline__ bool time_is_valid(double T) { return T >= 1 && T <= (double)OOB_DIST_MAX_T; }

__device__ __forceinline__ void refuse(const Args &a, long long i, int st) {
    a.status[i] = st;
    a.vx[2 * i] = 0; a.vx[2 * i + 1] = 0; a.slowest[i] = 0;
}

// A plan of more than kT templates, the first of them listed: what the first kT or the next one are refused for.
__device__ __forceinline__ void refuse_many(const Args &a, const double *s_tT, const unsigned *jx, long long i) {
    bool ok = true;
    for (int k = 0; k < kT; ++k) ok &= time_is_valid(s_tT[jx[k * kLanes] & 0xffff]);
    refuse(a, i, ok ? OOB_DIST_TOO_MANY_TEMPLATES : OOB_DIST_BAD_TIME);
}

// The distribution `ne` of a plan of t templates (none: it was refused), every entry of base and extra written once; or, with `open`, its list
// in rows 0 .. t-1.
__device__ __forceinline__ void write_rows(const Args &a, long long i, const unsigned *jx, const unsigned *ne, int t, bool open) {
    int k = 0;
    unsigned next = t == 0 ? a.p : open ? 0 : jx[0] & 0xffff, have = open ? jx[0] : ne[0];
    for (int j = 0; j < a.p; ++j) {
        unsigned w = 0;
        if ((unsigned)j == next) {
            w = have;
            ++k;
            const unsigned row = k < t ? jx[k * kLanes] : 0xffffu;
            next = open && k < t ? (unsigned)k : row & 0xffff;
            have = open ? row : k < t ? ne[k * kLanes] : 0;
        }
        a.base[(long long)j * a.capacity + i] = (unsigned short)w;
        a.extra[(long long)j * a.capacity + i] = (unsigned short)(w >> 16);
    }
}

// As write_rows, for a wave.
__device__ __forceinline__ void write_wave(const Args &a, long long i0, const unsigned *jx, const unsigned *ne, int t, bool open, unsigned *area) {
    const int lane = threadIdx.x & (kLanes - 1), r = lane >> 4;
    const long long at = r * a.capacity + i0 + 4 * (lane & 15);
    unsigned short *base = a.base + at, *extra = a.extra + at;
    u32x4 *const wide = (u32x4 *)area;
    int k = 0, next = t == 0 ? a.p : open ? 0 : (int)(jx[0] & 0xffff);
    unsigned have = open ? jx[0] : ne[0];
    for (int j0 = 0; j0 < a.p; j0 += kRows) {
#pragma unroll
        for (int h = 0; h < kRows / 4; ++h) wide[h * kLanes + lane] = (u32x4)0;
        wave_sync();
        while (next < std::min(j0 + kRows, a.p)) {
            area[(next - j0) * kLanes + lane] = have;
            ++k;
            const unsigned row = k < t ? jx[k * kLanes] : (unsigned)a.p;
            next = open && k < t ? k : (int)(row & 0xffff);
            have = open ? row : k < t ? ne[k * kLanes] : 0;
        }
        wave_sync();
#pragma unroll
        for (int h = 0; h < kRows / 4; ++h) {
            const u32x4 w = wide[h * kLanes + lane];
            if (j0 + 4 * h + r < a.p) {
                u32x2 lo, hi;
                lo.x = __builtin_amdgcn_perm(w.y, w.x, 0x05040100); hi.x = __builtin_amdgcn_perm(w.y, w.x, 0x07060302);
                lo.y = __builtin_amdgcn_perm(w.w, w.z, 0x05040100); hi.y = __builtin_amdgcn_perm(w.w, w.z, 0x07060302);
                *(u16x4 *)base = __builtin_bit_cast(u16x4, lo);
                *(u16x4 *)extra = __builtin_bit_cast(u16x4, hi);
            }
            base += 4 * a.capacity;
            extra += 4 * a.capacity;
        }
        wave_sync();
    }
}

// What one microbatch less for a fullest pipeline of n, or more for an emptiest one, costs a template at the level m2 / 2: the same double
// wherever it is formed (nothing is left to contraction).
__device__ __forceinline__ double cost_of_one(double T, int n, double m2, bool remove) {
    const double q = T * m2;
    return __builtin_fma(T * T, (double)(remove ? 1 - 2 * n : 2 * n + 1), remove ? q : -q);
}

// v >= 0, rounded to nearest: the highest 64 bits and whether anything is below them.
__device__ __forceinline__ double nearest(i128 v) {
    const unsigned long long hi = (unsigned long long)(v >> 64), lo = (unsigned long long)v;
    const int up = hi ? __clzll((long long)hi) : 64;
    unsigned long long top = lo;
    if (up < 64) top = (unsigned long long)(v >> (64 - up)) | (unsigned long long)(lo << up != 0);
    return ldexp((double)top, 64 - up);
}

// The template that one microbatch more or less costs least, the first of equals, among those whose cost in doubles is at most
// `near`.  ne: K words of this lane to work in.
template <int K>
__device__ __forceinline__ int exact_pick(const double *s_tT, const unsigned *jx, unsigned *ne, const int (&n)[K], const int (&e)[K], int t, long long mu,
                                          bool remove, double near) {
#pragma unroll
    for (int k = 0; k < K; ++k) ne[k * kLanes] = (unsigned)(n[k] + (remove && e[k] > 0));
    const long long s = remove ? 2 * mu : -2 * mu;
    long long Tp = 0;
    int mp = 0, pick = 0;
    i128 least = 0;
#pragma unroll 1
    for (int k = 0; k < t; ++k) {
        const int held = (int)ne[k * kLanes], m = remove ? 1 - 2 * held : 2 * held + 1;
        if (remove && held < 2) continue;
        const double T = s_tT[jx[k * kLanes] & 0xffff];
        if (T * T * m + T * (double)s > near) continue;
        const long long Tk = (long long)T;
        if (Tk == Tp && m == mp) continue; // twins
        const i128 v = (i128)Tk * (Tk * m + s); // |T m| and 2 mu are below 2^53
        if (Tp == 0 || v < least) { least = v; Tp = Tk; mp = m; pick = k; }
    }
    return pick;
}

// Plan i of t <= K templates by one lane, its templates in registers.  Template k has x pipelines; e of them hold n + 1
// microbatches, the others n (0 <= e < x): no division in the loops.  ne, best_ne: n | e << 16 of the allocation at hand and of the best.
//
// Mostly no exchange lies on the stretch, and then nothing has to be searched.  An exchange of a microbatch between two templates, taken from
// a fullest pipeline of d and given to an emptiest one of r, costs A + B with A = T_d^2 (1 - 2 n_d) + 2 T_d mu and B = T_r^2 (1 + 2 n_r)
// - 2 T_r mu.  If A + B > 0 for all T_d != T_r, the allocation is the only optimum at the level mu but for exchanges between templates of
// the same time (the problem is separable and convex: a strict minimum among its neighbours is the minimum).  Where that holds for the allocation
// of the stretch's middle at both ends of the stretch, the path has no exchange on the stretch (A + B <= 0 is what makes one pay) and is that
// allocation, or with twins (templates of the same time), which share their microbatches out in an order that hangs on the level, the
// allocation of the lower end.  Otherwise, and with twins, FOLLOW = true goes on from the lower end, and FOLLOW = false leaves the ends of
// the stretch in vx (a second allocation in the same loop takes 40 registers more than it has).
// mu, mu_hi: the ends of a stretch that is known (mu_hi = -1: it is not).  base and extra are the caller's.
enum { kRefused, kSolved, kOpen };
template <int K, bool FOLLOW>
__device__ __forceinline__ int solve(const Args &a, const double *s_tT, const unsigned *jx, unsigned *best_ne, unsigned *ne, long long i, int t,
                                     int xs, long long mu, long long mu_hi) {
    double T[K], inv[K];
    int x[K], n[K], e[K];
    int again = 0;
    auto inverse = [&](int k) { return s_tT[a.p + (jx[k * kLanes + again] & 0xffff)]; };
    bool valid = true, twins = false, exact = true, walk = FOLLOW && mu_hi >= 0, open = false;
    double H = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) { // no branch: the reads of all templates are in flight together
        const unsigned w = k < t ? jx[k * kLanes] : 0;
        T[k] = s_tT[w & 0xffff];
        inv[k] = s_tT[a.p + (w & 0xffff)];
        x[k] = (int)(w >> 16);
        n[k] = e[k] = 0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (k < t) {
            valid &= time_is_valid(T[k]);
            exact &= T[k] < kExactT;
            H += (double)x[k] * inv[k];
#pragma unroll
            for (int l = 0; l < k; ++l) twins |= T[l] == T[k];
        }
    if (!valid || t == 0 || xs > a.Q) {
        refuse(a, i, !valid ? OOB_DIST_BAD_TIME : t == 0 ? OOB_DIST_NO_PIPELINE : OOB_DIST_TOO_FEW_MICROBATCHES);
        return kRefused;
    }
    const double mean = H / xs, L0 = (double)a.Q / H;
    double D = 0;
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (k < t) {
            const double r = inv[k] - mean;
            D += r * r * x[k];
        }
    if (!walk) mu = (long long)(L0 + 0.5);
    // D is formed here, the reciprocals are read again and x converted again where they are used: registers decide how many waves run
    asm volatile("" : "+v"(D), "+v"(again));
#pragma unroll
    for (int k = 0; k < K; ++k) asm volatile("" : "+v"(x[k]));

    // every exchange between templates of different times costs at level mu (see above)
    auto settled = [&](double mu) {
        const double m2 = 2.0 * mu;
        double a1 = kHuge, a2 = kHuge, b1 = kHuge, b2 = kHuge; // smallest A and B, and smallest of another time, less their rounding
        double at = 0, bt = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k < t) {
                const int full = n[k] + (e[k] > 0);
                const double sq = T[k] * T[k], q = T[k] * m2, pa = sq * (2 * full - 1), pb = sq * (2 * n[k] + 1);
                const double A = full < 2 ? kHuge : (q - pa) - (q + pa) * kEps, B = (pb - q) - (pb + q) * kEps;
                a2 = T[k] == at ? a2 : fmin(a2, fmax(a1, A));
                at = A < a1 ? T[k] : at;
                a1 = fmin(a1, A);
                b2 = T[k] == bt ? b2 : fmin(b2, fmax(b1, B));
                bt = B < b1 ? T[k] : bt;
                b1 = fmin(b1, B);
            }
        return (at != bt ? a1 + b1 : fmin(a1 + b2, a2 + b1)) > 0.0;
    };
    long long S1; // below 2^51
    i128 S2, best;
    for (;;) { // at the middle of the stretch, then (walk) at its lower end
#pragma unroll
        for (int k = 0; k < K; ++k) asm volatile("" : "+v"(T[k])); // products of the times are formed here, not kept for the next round
        // the optimum at the level mu: rounded, then one microbatch more or less where that is cheapest (the first of equals)
        const double m2 = 2.0 * (double)mu;
        int tot = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
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
            double c[K], most = 0; // what one microbatch less or more costs a template; what their rounding can come to
#pragma unroll
            for (int k = 0; k < K; ++k) {
                c[k] = kHuge;
                if (k < t) {
                    if (!remove || n[k] >= 2) c[k] = cost_of_one(T[k], n[k], m2, remove);
                    most = fmax(most, 4.0 * kEps * (T[k] * m2 + T[k] * T[k] * (2 * n[k] + 1)));
                }
            }
            for (;;) {
                double c1 = kHuge, c2 = kHuge;
                int pick = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    c2 = fmin(c2, fmax(c1, c[k]));
                    pick = c[k] < c1 ? k : pick;
                    c1 = fmin(c1, c[k]);
                }
                if (c1 >= kHuge) break; // cannot happen: tot > Q >= pipelines, so some pipeline holds two
                if (c2 - c1 <= most && !exact) { // templates of one time have the same double for the same cost
                    const double Tp = s_tT[jx[pick * kLanes] & 0xffff];
                    bool mixed = false;
#pragma unroll
                    for (int k = 0; k < K; ++k) mixed |= c[k] - c1 <= most && T[k] != Tp;
                    if (mixed) pick = exact_pick(s_tT, jx, best_ne, n, e, t, mu, remove, c1 + most);
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (k != pick) continue;
                    // its pipelines that are alike cost alike: all of them, as far as there are microbatches to move, in one step (one by one
                    // 3 500 cycles more of a wave's 11 300)
                    int move;
                    bool next; // the template's pipelines start over: another cost
                    if (remove) { // the fullest ones give one each
                        if (e[k] == 0) { --n[k]; e[k] = x[k]; }
                        move = std::min(tot - a.Q, e[k]);
                        e[k] -= move;
                        next = e[k] == 0;
                        tot -= move;
                    } else {      // the emptiest ones take one each
                        move = std::min(a.Q - tot, x[k] - e[k]);
                        e[k] += move;
                        next = e[k] == x[k];
                        if (next) { ++n[k]; e[k] = 0; }
                        tot += move;
                    }
                    if (next) { // formed anew: sums of steps would add up their roundings
                        double Tk = T[k];
                        asm volatile("" : "+v"(Tk));
                        c[k] = remove && n[k] < 2 ? kHuge : cost_of_one(Tk, n[k], 2.0 * (double)mu, remove);
                        most = fmax(most, 4.0 * kEps * (Tk * (2.0 * (double)mu) + Tk * Tk * (2 * n[k] + 1)));
                    }
                }
                if (tot == a.Q) break;
            }
        }
        {
            // S1 = sum_i N_i T_i and S2 = sum_i (N_i T_i)^2, exactly: all of it is integers in doubles.  sum_i N_i = Q < 2^16, so S1 < 2^51, w = sum N_i^2 of
            // a template and their sum are at most 2^32 and S2 at most 2^102.  A product and what its rounding left out (by fma) are two instructions, a sum and
            // what its rounding left out (two-sum) six; a part left out of T^2 is below 2^16, of T^2 w or of a sum at most 2^48, so that all of
            // them together, at most 16 templates, come to 2^53 at most.  In 128-bit integers a template takes 60 instructions, a third of them
            // products at a quarter of the rate, here 25.
#pragma clang fp contract(off)
            double sum = 0, rest = 0, s1 = 0;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (k < t) {
                    const double N = (double)n[k], E = (double)e[k], X = (double)x[k];
                    const double w = __builtin_fma(N * N, X, __builtin_fma(2.0, N, 1.0) * E);
                    s1 = __builtin_fma(T[k], __builtin_fma(N, X, E), s1);
                    const double sq = T[k] * T[k], v = sq * w, to = sum + v, part = to - sum;
                    rest += __builtin_fma(__builtin_fma(T[k], T[k], -sq), w, __builtin_fma(sq, w, -v));
                    rest += (sum - (to - part)) + (v - part);
                    sum = to;
                }
            const double high = floor(sum * 0x1p-52);
            S1 = (long long)s1;
            S2 = ((i128)(long long)high << 52) + (long long)__builtin_fma(-0x1p52, high, sum) + (long long)rest;
        }
        best = (i128)xs * S2 - (i128)S1 * S1;
        if (walk) break;
        const double V = nearest(best) / (double)xs; // sum of squared deviations of a feasible allocation
        // with twins the distribution met first among equal ones depends on where the path starts: it starts where the
        // cruder bound, sqrt(V), puts it
        const double narrow = twins ? 1.0 : fmin(sqrt(D) / H, 1.0);
        const double R = sqrt(V) * (narrow * (1.0 + 1e-9) + 1e-12) + L0 * 1e-9 + 2.0; // widened for the rounding of these few operations
        mu = L0 - R > 0 ? (long long)(L0 - R) : 0;
        mu_hi = (long long)(L0 + R) + 1;
        bool only = true; // one end after the other: together they take more registers than the kernel has
#pragma unroll 1
        for (int side = 0; side < 2; ++side) only &= settled(side ? (double)mu_hi : (double)mu);
        if (only && !twins) break;
        if constexpr (!FOLLOW) { open = true; break; }
        walk = true;
    }
    double slow = 0; // a pipeline's time is below 2^51
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (k < t) {
            best_ne[k * kLanes] = (unsigned)n[k] | (unsigned)e[k] << 16;
            slow = fmax(slow, T[k] * (double)(n[k] + (e[k] > 0)));
        }
    if constexpr (FOLLOW) {
#pragma unroll
        for (int k = 0; k < K; ++k) // the allocation once more in LDS, for the templates that give
            if (walk && k < t) ne[k * kLanes] = (unsigned)n[k] | (unsigned)e[k] << 16;
        while (walk && !settled((double)mu_hi)) {
            // the next exchange: a microbatch of a fullest pipeline of template d (n_d of them) goes to an emptiest
            // pipeline of a slower template r (n_r): it pays from the level c / w on,
            // c = T_d^2 + T_r^2 - 2 T_d^2 n_d + 2 T_r^2 n_r,  w = 2 (T_r - T_d) > 0; the first of the smallest levels
            int bd = -1, br = -1;
            double bc = 0, be = 0, bw = 1;
            bool near = false;
            for (int d = 0; d < t; ++d) {
                const unsigned wd = ne[d * kLanes];
                const int nd = (int)(wd & 0xffff) + (wd >> 16 ? 1 : 0);
                const double Td = s_tT[jx[d * kLanes] & 0xffff], cd = Td * Td * (1 - 2 * nd);
                if (nd < 2) continue;
#pragma unroll
                for (int r = 0; r < K; ++r) {
                    const double Tr = T[r];
                    if (r >= t || Tr <= Td) continue;
                    const double cr = Tr * Tr * (1 + 2 * n[r]), c = cd + cr, w = 2.0 * (Tr - Td); // w exact
                    const double err = (cr - cd) * kEps, diff = c * bw - bc * w;
                    near |= bd >= 0 && fabs(diff) <= 2.0 * (err * bw + be * w);
                    if (bd < 0 || diff < 0) { bc = c; be = err; bw = w; bd = d; br = r; }
                }
            }
            if (near && !exact) { // once more, exactly, among those that the rounding does not put above the smallest
                const double mc = bc, me = be, mw = bw;
                i128 xc = 0;
                long long xw = 1;
                bd = -1;
                for (int d = 0; d < t; ++d) {
                    const unsigned wd = ne[d * kLanes];
                    const int nd = (int)(wd & 0xffff) + (wd >> 16 ? 1 : 0);
                    const double Td = s_tT[jx[d * kLanes] & 0xffff], cd = Td * Td * (1 - 2 * nd);
                    if (nd < 2) continue;
                    unsigned hits = 0;
#pragma unroll
                    for (int r = 0; r < K; ++r) {
                        const double Tr = T[r];
                        if (r >= t || Tr <= Td) continue;
                        const double cr = Tr * Tr * (1 + 2 * n[r]), c = cd + cr, w = 2.0 * (Tr - Td);
                        if (c * mw - mc * w <= 2.0 * ((cr - cd) * kEps * mw + me * w)) hits |= 1u << r;
                    }
                    for (; hits; hits &= hits - 1) {
                        const int r = __ffs((int)hits) - 1;
                        const long long kd = (long long)Td, kr = (long long)s_tT[jx[r * kLanes] & 0xffff], ew = kr - kd; // below 2^36
                        const i128 ec = (i128)kd * (kd * (1 - 2 * nd)) + (i128)kr * (kr * (1 + 2 * (int)(ne[r * kLanes] & 0xffff)));
                        if (bd < 0 || ec * xw < xc * ew) { xc = ec; xw = ew; bd = d; br = r; }
                    }
                }
            }
            if (bd < 0) break;
            const unsigned xd = jx[bd * kLanes], xr = jx[br * kLanes];
            const long long Td = (long long)s_tT[xd & 0xffff], Tr = (long long)s_tT[xr & 0xffff];
            unsigned wd = ne[bd * kLanes], wr = ne[br * kLanes];
            const int nd = (int)(wd & 0xffff) + (wd >> 16 ? 1 : 0), nr = (int)(wr & 0xffff);
            const i128 change = (i128)Tr * Tr * (2 * nr + 1) - (i128)Td * Td * (2 * nd - 1);
            if (change > (i128)(2 * (Tr - Td)) * mu_hi) break; // past the stretch
            S1 += Tr - Td;
            S2 += change;
            wd = wd >> 16 ? wd - 0x10000u : (wd - 1) | ((xd >> 16) - 1) << 16;   // a fullest pipeline gives
            wr = (wr >> 16) + 1 == xr >> 16 ? (wr & 0xffff) + 1 : wr + 0x10000u; // an emptiest one takes
            ne[bd * kLanes] = wd;
            ne[br * kLanes] = wr;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k == bd) { n[k] = (int)(wd & 0xffff); e[k] = (int)(wd >> 16); }
                if (k == br) { n[k] = (int)(wr & 0xffff); e[k] = (int)(wr >> 16); }
            }
            const i128 v = (i128)xs * S2 - (i128)S1 * S1;
            if (v < best) {
                best = v;
                slow = 0;
                for (int k = 0; k < t; ++k) {
                    const unsigned w = ne[k * kLanes];
                    best_ne[k * kLanes] = w;
                    slow = fmax(slow, s_tT[jx[k * kLanes] & 0xffff] * (double)((w & 0xffff) + (w >> 16 ? 1 : 0)));
                }
            }
        }
    }
    if (open) {
        a.vx[2 * i] = (unsigned long long)mu;
        a.vx[2 * i + 1] = (unsigned long long)mu_hi;
        return kOpen;
    }
    a.status[i] = OOB_DIST_OK;
    a.vx[2 * i] = (unsigned long long)best;
    a.vx[2 * i + 1] = (unsigned long long)(best >> 64);
    a.slowest[i] = (long long)slow;
    return kSolved;
}

// The times, [p], then [p] reciprocals; first: that of the thread's number.
__device__ __forceinline__ void load_times(const Args &a, double *s_tT, long long first) {
    for (int j = threadIdx.x; j < a.p; j += blockDim.x) {
        const double T = (double)(j < (int)blockDim.x ? first : a.tT[j]); // exact where it is used (up to 2^35)
        s_tT[j] = T;
        s_tT[a.p + j] = 1.0 / T;
    }
    __syncthreads();
}

// The first of two launches: the plans that cannot be solved and those of at most kFew templates, with FOLLOW = false only where no exchange
// lies on the stretch.  The others get a mark in `status`, kMarked + templates << 8 + rank among the workgroup's plans of at most kFew
// templates, or of more; where base and extra can hold it, their list stands there (with the counts read once more the second launch took
// 170 us instead of 85).
constexpr int kMarked = 1 << 30;
template <bool FOLLOW> __global__ void __launch_bounds__(kFirstThreads, FOLLOW ? 3 : 4) k_dist_first(Args a) {
    constexpr int W = (kT + kFew + (FOLLOW ? kFew : kRows)) * kLanes;
    static_assert(kFew >= kRows, "rows of the wave where its allocations were");
    HIP_DYNAMIC_SHARED(double, s_tT)
    __shared__ __attribute__((aligned(16))) unsigned s_words[kFirstThreads / kLanes * W]; // of a wave: lists, best and current allocations
    __shared__ int s_ranks[2];
    if (threadIdx.x < 2) s_ranks[threadIdx.x] = 0;
    const long long i = (long long)blockIdx.x * kFirstThreads + threadIdx.x;
    const int lane = threadIdx.x & (kLanes - 1);
    const bool whole = i - lane + kLanes <= a.count; // the same for a wave
    unsigned *const words = s_words + threadIdx.x / kLanes * W, *const area = words + (kT + kFew) * kLanes;
    unsigned *const jx = words + lane, *const best_ne = jx + kT * kLanes;
    int xs = 0, t = 0, got = kRefused;
    const long long first = threadIdx.x < a.p ? a.tT[threadIdx.x] : 0; // on its way while the templates are listed
    if (whole) t = list_wave(a, i - lane, jx, words + (kT + 1) * kLanes, &xs);
    else if (i < a.count) t = list_templates(a, i, jx, kT, &xs);
    load_times(a, s_tT, first);
    if (i >= a.count) return;
    if (t <= kFew) got = solve<kFew, FOLLOW>(a, s_tT, jx, best_ne, area + lane, i, t, xs, 0, -1);
    else if (t > kT) refuse_many(a, s_tT, jx, i);
    else got = kOpen;
    const bool left = got == kOpen;
    if (a.lists && whole) write_wave(a, i - lane, jx, left ? jx : best_ne, got == kRefused ? 0 : t, left, area);
    else if (a.base && (a.lists || !left)) write_rows(a, i, jx, left ? jx : best_ne, got == kRefused ? 0 : t, left);
#pragma unroll
    for (int kind = 0; kind < 2; ++kind) { // a wave's places in one step
        const bool mine = left && (t > kFew) == kind;
        const unsigned long long m = __ballot(mine);
        int rank = 0;
        if (m && lane == __ffsll((long long)m) - 1) rank = atomicAdd(&s_ranks[kind], __popcll(m));
        if (m) rank = __shfl(rank, __ffsll((long long)m) - 1) + __popcll(m & ((1ull << lane) - 1));
        if (mine) a.status[i] = kMarked + (t << 8) + rank;
    }
}

// The only launch for few plans: all of them, 64 to a wave.
__global__ void __launch_bounds__(kLanes, 2) k_dist_once(Args a) {
    constexpr int W = kT * kLanes;
    HIP_DYNAMIC_SHARED(double, s_tT)
    __shared__ __attribute__((aligned(16))) unsigned s_words[3 * W]; // lists, best and current allocations
    const int lane = threadIdx.x;
    const long long i = (long long)blockIdx.x * kLanes + lane;
    unsigned *const jx = s_words + lane;
    const bool whole = i - lane + kLanes <= a.count;
    int xs = 0, t = 0, got = kRefused;
    const long long first = lane < a.p ? a.tT[lane] : 0; // on its way while the templates are listed
    if (whole) t = list_wave(a, i - lane, jx, s_words + 2 * W, &xs);
    else if (i < a.count) t = list_templates(a, i, jx, kT, &xs);
    load_times(a, s_tT, first);
    if (i >= a.count) return;
    if (t > kT) refuse_many(a, s_tT, jx, i);
    else if (t <= kFew) got = solve<kFew, true>(a, s_tT, jx, jx + W, jx + 2 * W, i, t, xs, 0, -1);
    if (t > kFew && t <= kT) got = solve<kT, true>(a, s_tT, jx, jx + W, jx + 2 * W, i, t, xs, 0, -1);
    if (a.base && whole) write_wave(a, i - lane, jx, jx + W, got == kRefused ? 0 : t, false, s_words + 2 * W);
    else if (a.base) write_rows(a, i, jx, jx + W, got == kRefused ? 0 : t, false);
}

// The list of t <= K templates that the first launch left for plan i, read where it is, or from the counts.  Returns the pipelines.
template <int K> __device__ __forceinline__ int listed(const Args &a, long long i, unsigned *jx, int t) {
    int xs = 0;
    if (a.lists) {
        unsigned v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = k < t ? (unsigned)a.base[k * a.capacity + i] | (unsigned)a.extra[k * a.capacity + i] << 16 : 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            jx[k * kLanes] = v[k];
            xs += (int)(v[k] >> 16);
        }
    } else {
        list_templates(a, i, jx, K, &xs);
    }
    return xs;
}

// A marked plan whose list has been read: solved, its distribution written.  From a list the entries that hold none of it are zeros.
template <int K>
__device__ __forceinline__ void solve_listed(const Args &a, const double *s_tT, const unsigned *jx, unsigned *best_ne, unsigned *ne, long long i, int t,
                                             int xs, long long mu, long long mu_hi) {
    const int got = solve<K, true>(a, s_tT, jx, best_ne, ne, i, t, xs, mu, mu_hi);
    if (a.lists && got != kRefused) {
        for (int k = 0; k < t; ++k) a.base[k * a.capacity + i] = a.extra[k * a.capacity + i] = 0;
        for (int k = 0; k < t; ++k) {
            const unsigned w = best_ne[k * kLanes];
            const long long at = (long long)(jx[k * kLanes] & 0xffff) * a.capacity + i;
            a.base[at] = (unsigned short)w;
            a.extra[at] = (unsigned short)(w >> 16);
        }
    } else if (a.base) {
        write_rows(a, i, jx, best_ne, got == kRefused ? 0 : t, false);
    }
}

// The second launch: the marked ones of `span` consecutive plans, side by side, those of few templates and then the others.  `slices` waves, `spans`
// workgroups apart, share a span: a wave has the plans whose rank / ranks is its slice modulo `slices`.  Who has a plan depends on its mark
// alone, and nobody else writes that: the marks of others may be there or gone.
__global__ void __launch_bounds__(kLanes, 2) k_dist_rest(Args a, int span, int spans, int slices) {
    HIP_DYNAMIC_SHARED(double, s_tT) // the times, then [span] 16-bit numbers of plans: few templates from the front, many from the back
    __shared__ unsigned s_words[3 * kT * kLanes]; // lists, best and current allocations
    unsigned short *const marked = (unsigned short *)(s_tT + 2 * a.p);
    const int lane = threadIdx.x, slice = blockIdx.x / spans, ranks = kLanes * kFirstThreads / span;
    const long long i0 = (long long)(blockIdx.x - slice * spans) * span;
    const unsigned long long below = (1ull << lane) - 1;
    const long long first = lane < a.p ? a.tT[lane] : 0;
    int few = 0, many = 0;
    for (int o0 = 0; o0 < span; o0 += kLanes * kScan) {
        int st[kScan];
#pragma unroll
        for (int q = 0; q < kScan; ++q) {
            const long long i = i0 + o0 + q * kLanes + lane;
            st[q] = i < a.count ? a.status[i] : 0;
        }
#pragma unroll
        for (int q = 0; q < kScan; ++q) {
            const int t = st[q] >> 8 & 31;
            const bool mine = st[q] >= kMarked && (st[q] & 255) / ranks % slices == slice;
            const unsigned long long mf = __ballot(mine && t <= kFew), mm = __ballot(mine && t > kFew);
            const unsigned short w = (unsigned short)((o0 + q * kLanes + lane) | t << kSpanBits);
            if (mine) marked[t <= kFew ? few + __popcll(mf & below) : span - 1 - many - __popcll(mm & below)] = w;
            few += __popcll(mf);
            many += __popcll(mm);
        }
    }
    if (few + many == 0) return; // uniform
    load_times(a, s_tT, first);
    unsigned *const jx = s_words + lane, *const best_ne = jx + kT * kLanes, *const ne = best_ne + kT * kLanes;
    for (int q = lane; q < few; q += kLanes) {
        const int w = marked[q], t = w >> kSpanBits;
        const long long i = i0 + (w & ((1 << kSpanBits) - 1));
        const int xs = listed<kFew>(a, i, jx, t);
        solve_listed<kFew>(a, s_tT, jx, best_ne, ne, i, t, xs, (long long)a.vx[2 * i], (long long)a.vx[2 * i + 1]);
    }
    for (int q = lane; q < many; q += kLanes) {
        const int w = marked[span - 1 - q], t = w >> kSpanBits;
        const long long i = i0 + (w & ((1 << kSpanBits) - 1));
        const int xs = listed<kT>(a, i, jx, t);
        solve_listed<kT>(a, s_tT, jx, best_ne, ne, i, t, xs, 0, -1);
    }
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
    const size_t times = 2 * (size_t)p * sizeof(double);
    hipStream_t st = (hipStream_t)stream;
    if (count <= kOnce) {
        a.lists = 0;
        hipLaunchKernelGGL(k_dist_once, dim3((unsigned)((count + kLanes - 1) / kLanes)), dim3(kLanes), times, st, a);
    } else {
        a.lists = base && apart(x, base, p, capacity) && apart(x, extra, p, capacity) && apart(base, extra, p, capacity);
        const bool follow = count <= kFollow;
        const int span = follow ? kFirstThreads : 1 << kSpanBits;
        const long long spans = (count + span - 1) / span;
        const int slices = (int)std::min<long long>(span / kLanes, std::max(1ll, kRestWaves / spans));
        hipLaunchKernelGGL(follow ? k_dist_first<true> : k_dist_first<false>, dim3((unsigned)((count + kFirstThreads - 1) / kFirstThreads)),
                           dim3(kFirstThreads), times, st, a);
        hipLaunchKernelGGL(k_dist_rest, dim3((unsigned)(spans * slices)), dim3(kLanes), times + span * sizeof(unsigned short), st, a, span, (int)spans, slices);
    }
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
