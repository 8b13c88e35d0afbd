// Exact minimum of the pipeline cost (Section 4.1.2 of the Oobleck paper; the closed form of
// Eq. 1-4) over all explicit pipelines, for gfx950.
//
// With k* the first slowest stage and tau its time,
//     C = sum_{i<k*} t_i + N_b tau + sum_{i>k*} (2 t_i - tau)                        (N_b given)
//     C = sum_{i<k*} (t_i + 4 tau) + 4 tau + sum_{i>k*} (2 t_i + 3 tau)              (N_b = 4 S)
// so around a FIXED slowest stage (u, v, d) the stages before and after it are two independent
// shortest-path problems.  A stage never crosses a node boundary and the stages fill node after
// node, so a pipeline around (u, v, d) is: `a` whole nodes covering layers [0, q), then g GPUs of the
// slowest stage's node covering [q, u), the stage itself, the remaining h = M - g - d GPUs of that
// node covering [v, x), and b whole nodes covering [x, L); n = a + 1 + b.
//
// Branch and bound over the slowest stage.  Of the tens of thousands of possible slowest stages a
// few hundred can be the slowest stage of a minimum: a stage much slower than the best pipeline's is
// too dear, a much faster one leaves the other layers too few GPUs.  Four launches find them:
//   k_exact_prep    validates the profile, forms the prefix sums and lists the possible slowest stages
//                   in ascending order of their time (counting sort over the leading bits of the double);
//   k_exact_bounds  per bucket of consecutive entries of that list and per template n a lower bound of
//                   the cost around each of them: GPUs and stages are priced (Lagrangian multipliers
//                   lambda per GPU, mu per stage where the stage limit binds) instead of counted, which
//                   leaves two one-dimensional shortest paths per bucket, side and multiplier;
//   k_exact_eval<kFirst>  evaluates the most promising slowest stages of every template exactly;
//   k_exact_filter        keeps those whose bound does not exceed what was found;
//   k_exact_eval<kRest>   evaluates these exactly, looking at the bounds again as the minima fall.
// Small jobs (kDirectMax) skip the bounds and evaluate every stage but those too dear by their time alone.
// Measured, one call: 98 layers, 8 GPUs per node, 57 templates 20.4 -> 0.39 ms (2 000 evaluations of 17 524 slowest stages);
// 26 layers, 4 GPUs per node, N_b = 4 S 171 -> 54 us; 48 layers, 8 GPUs per node, N_b = 20 with
// the limit binding 38.0 -> 0.54 ms (the evaluation of every stage in tables of the workspace before).
//
// k_exact_eval: one workgroup per slowest stage, everything in LDS and registers, times as exact integers in doubles.
// Phase 1, per wave, no workgroup barrier: the one-node table of start layer q, G_q[r][g] = least cost
// of covering r layers from q on with stages on exactly g GPUs of one node (in registers, or row after row in LDS); it yields W[r][q] =
// G_q[r][M] (a whole node) and GU[r][g] = G_{u-r}[r][g].  Phase 2: the node-level recurrence
// NP_{a+1}[p] = min_r NP_a[p-r] + W[r][p-r], one barrier per node count.  The same for the layers after v,
// mirrored, side by side with it; then every (template, a, g) combination.  Stages slower than tau are
// no use, so a node covers at most a few layers: all loops are bounded by that band.
// With the stage count as a further index (oob_exact_minimum_staged where the limit S <= N_b can bind) the tables
// hold plain sums of t per number of stages and the coefficient of tau follows from the counts at the end.
//
// k_exact_flat (tables in the caller's workspace, int64): the plain recurrence over (layer, GPUs
// used [, stages used]).  It serves shapes whose tables exceed LDS and times beyond 2^52.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <type_traits>

#include "oob_exact.h"
#include "oob_exact_sizes.h"
#include "oob_layout.h"

namespace oob_exact {

using oob::wg_sync;

constexpr int kThreads = 256;    // k_exact_flat
constexpr int kFlatSlots = 2048; // its workgroups in flight at most, each with tables of its own
constexpr long long kInf = 1ll << 61;
constexpr long long kForbidden = 1ll << 62;
constexpr long long kDoubleExact = 1ll << 52;
constexpr double kNone = __builtin_huge_val();
constexpr unsigned long long kNoneBits = 0x7FF0000000000000ull;

constexpr int kPrepThreads = 1024;
constexpr int kBoundThreads = 576;   // eight waves for the paths, one for the fewest nodes
constexpr int kFirst = 1, kRest = 2, kAll = 0;

struct Args {
    oob_profile prof;
    int L, M, n_min, n_max, Nb, Dmax, Smax, fast, staged, bounds;
    int sums;             // the profile without the ends of the stages (EvalLds)
    int eval_pad, bounds_pad; // rows of the profile in LDS padded (Prof)
    int regs;                 // k_exact_eval holds the tables of a node in registers where it can
    int nodes;            // min(n_max, L): more nodes than layers make no pipeline
    int top, live;        // last template that can get a minimum (answered(), nodes), number of templates up to it
    long long cap;
    long long limit;      // every cost must stay below this (2^52 for the LDS path, 2^61 otherwise)
    Head *head;
    long long *PT;        // [(L+1) M] prefix sums of F + B for d GPUs: entry l M + d-1, forbidden entries left out
    unsigned char *flo;   // [(L+1) M] first layer u for which [u, v) may run on d GPUs of a node (memory, forbidden counts)
    double *ctau;         // [ncand] possible slowest stages, ascending (by bins): time
    unsigned *cuvd;       //         u | v << 8 | d << 16
    int nk;               // pairs of multipliers
    float *lb;            // [ncand][nk] lower bounds but for the part that depends on the template
    double *blo;          // [nbuckets] fastest stage of a bucket, the unit of its multipliers
    int *bfew;            // [nbuckets] fewest nodes that can cover the layers
    float *blb;           // [nbuckets][count] smallest bound of a bucket
    unsigned short *barg; // [nbuckets][count] and the entry it belongs to, from the first of the bucket
    unsigned *list;       // [ncand] entries left to evaluate
    unsigned *over;       // [ncand] entries that k_exact_flat has to evaluate (tables with stage counts beyond LDS)
    long long *slots;     // k_exact_flat: [slots][2][(L+1)][(Dmax+1)][J]
    unsigned long long *best; // per template: smallest cost so far
    int *status;
};


// Whether the template for n nodes gets a minimum: without stage counts not where the stage limit can bind.  The others'
// best stays infinite, and no bound, pick or evaluation is for them.
__device__ __forceinline__ bool answered(const Args &a, int n) { return a.staged || a.Nb == 0 || a.Nb >= imin(a.L, n * a.M); }

// ---- what one workgroup's last act is: hand the minima to the caller ------------------------------
// Results as int64: -1 where no pipeline exists, -2 (unstaged entry point) where the stage limit
// can bind, so that the minimum without it is not the answer.
__device__ void finish(const Args &a, bool from_double) {
    for (int i = threadIdx.x; i <= a.n_max - a.n_min; i += blockDim.x) {
        const int n = a.n_min + i;
        const unsigned long long b = __hip_atomic_load(&a.best[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        long long out;
        if (!answered(a, n)) out = -2;
        else if (from_double) { const double x = __longlong_as_double((long long)b); out = x < kNone ? (long long)x : -1; }
        else out = (long long)b >= kInf / 2 ? -1 : (long long)b;
        ((long long *)a.best)[i] = out;
    }
}
// True in every thread of the workgroup that finishes last of the grid's (which all call this once).  What the
// others hand over are atomics on `best`, performed at the point where the last one reads them: waiting for the own ones
// orders them, no cache has to be written back (a release at agent scope, once per workgroup, cost more than the work
// of small jobs).
__device__ bool last_workgroup(const Args &a) {
    __shared__ unsigned s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wg_sync();
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(&a.head->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    wg_sync();
    return s_last != 0;
}

// ---------------------------------------------------------------------------------------------
// Preparation, one workgroup.  Validates the magnitudes: every cost is at most mult * w, w = the sum over
// the layers of the slowest allowed F + B of the layer plus its boundary term (a bound on the sum
// of all stage times of any pipeline), mult = N_b + 2 (4 S_max + 2 when N_b = 4 S).  status =
// OOB_EOVERFLOW unless that stays below the limit of the path; OOB_EINVAL for a negative entry.
// One launch in place of four (62 + 13 + 4 + 4 us at 98 layers x 8 GPUs): prefix sums instead of a table of all stage
// times, 37 us there and 12 us at 26 x 4, most of it the two walks over the layer pairs with LDS atomics.  (45 and 14 us with the
// list scattered to memory, the sums as integers that every stage turned into a double, and a lane per single layer at
// one LDS word for the fastest.)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long scan_add(unsigned long long x, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}
__device__ __forceinline__ int scan_max(int x, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x = imax(x, y);
    }
    return x;
}
// Triple i -> (u, v, d), u < v, d fastest, then u.
__device__ __forceinline__ void triple(int i, int M, int *u, int *v, int *d) {
    const int p = i / M;
    *d = i - p * M + 1;
    int w = (int)((sqrtf(8.0f * (float)p + 1.0f) + 1.0f) * 0.5f);
    while (w * (w - 1) / 2 > p) --w;
    while (w * (w + 1) / 2 <= p) ++w;
    *v = w;
    *u = p - w * (w - 1) / 2;
}

__global__ void __launch_bounds__(kPrepThreads) k_exact_prep(Args a, int room) {
    HIP_DYNAMIC_SHARED(long long, s_prep) // [(L+1)] bytes, [(L+1) M] times where the fast path needs them, then bytes, [room] entries of the list
    __shared__ int s_hist[kBins];
    __shared__ int s_bad, s_wave[kPrepThreads / 64];
    __shared__ unsigned long long s_sum[kPrepThreads / 64], s_min;
    const int L = a.L, M = a.M, W = L + 1, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
    const long long *fwd = (const long long *)a.prof.fwd_ns, *bwd = (const long long *)a.prof.bwd_ns;
    const long long *mem = (const long long *)a.prof.mem_bytes, *bnd = (const long long *)a.prof.boundary_ns;
    unsigned long long *s_pm = (unsigned long long *)s_prep;
    double *s_pt = (double *)(s_prep + W); // (read only where every one is an exact integer)
    unsigned char *s_lf = (unsigned char *)(s_pt + (a.fast ? (size_t)W * M : 0));
    unsigned *s_list = (unsigned *)(s_lf + ((size_t)W * M + 3) / 4 * 4);
    const int count = a.n_max - a.n_min + 1;
    for (int i = tid; i < count; i += blockDim.x) a.best[i] = kNoneBits; // +inf as a double, huge as an integer
    for (int i = tid; i < kBins; i += blockDim.x) s_hist[i] = 0;
    if (tid == 0) { s_bad = 0; s_min = kNoneBits; }
    wg_sync();
    // magnitudes and signs
    unsigned long long acc = 0;
    bool bad = false;
    for (int l = tid; l < L; l += blockDim.x) {
        long long worst = 0;
        for (int d = 0; d < M; ++d) {
            const long long f = fwd[(size_t)l * M + d], b = bwd[(size_t)l * M + d];
            bad = bad || f < 0 || b < 0;
            if (f < 0 || b < 0 || f >= kForbidden || b >= kForbidden) continue;
            const long long fb = (f >= kInf || b >= kInf) ? kInf : f + b;
            worst = fb > worst ? fb : worst;
        }
        const long long x = bnd[l];
        bad = bad || x < 0 || mem[l] < 0;
        if (x > 0) worst = (x >= kInf || worst >= kInf) ? kInf : worst + x;
        acc = acc + (unsigned long long)worst;
        if (acc > (unsigned long long)kInf) acc = (unsigned long long)kInf;
    }
    if (bad) s_bad = 1;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        acc += __shfl_xor(acc, d, 64);
        if (acc > (unsigned long long)kInf) acc = (unsigned long long)kInf;
    }
    if (lane == 0) s_sum[wave] = acc;
    // prefix sums, one wave per GPU count; wave nw - 1 also takes the bytes
    for (int d = wave; d < M; d += nw) {
        unsigned long long carry = 0;
        int last = 0; // first layer after the last forbidden one so far
        if (lane == 0) { a.PT[d] = 0; if (a.fast) s_pt[d] = 0; s_lf[d] = 0; }
        for (int l0 = 0; l0 < L; l0 += 64) {
            const int l = l0 + lane;
            const long long f = l < L ? fwd[(size_t)l * M + d] : 0, b = l < L ? bwd[(size_t)l * M + d] : 0;
            const bool forb = f >= kForbidden || b >= kForbidden;
            const unsigned long long x = scan_add(forb ? 0ull : (unsigned long long)f + (unsigned long long)b, lane) + carry;
            const int lf = imax(scan_max(forb ? l + 1 : 0, lane), last);
            if (l < L) {
                a.PT[(size_t)(l + 1) * M + d] = (long long)x;
                if (a.fast) s_pt[(size_t)(l + 1) * M + d] = (double)(long long)x;
                s_lf[(size_t)(l + 1) * M + d] = (unsigned char)lf;
            }
            carry = __shfl(x, 63, 64);
            last = __shfl(lf, 63, 64);
        }
    }
    if (wave == nw - 1) {
        unsigned long long carry = 0;
        if (lane == 0) s_pm[0] = 0;
        for (int l0 = 0; l0 < L; l0 += 64) {
            const int l = l0 + lane;
            const unsigned long long x = scan_add(l < L ? (unsigned long long)mem[l] : 0ull, lane) + carry;
            if (l < L) s_pm[l + 1] = x;
            carry = __shfl(x, 63, 64);
        }
    }
    wg_sync();
    unsigned long long w = 0;
    for (int i = 0; i < nw; ++i) { w += s_sum[i]; if (w > (unsigned long long)kInf) w = (unsigned long long)kInf; }
    const long long mult = (a.Nb > 0 ? (long long)a.Nb : 4ll * a.Smax) + 2;
    const int st = s_bad ? OOB_EINVAL : (long long)w >= a.limit / mult ? OOB_EOVERFLOW : OOB_OK;
    const bool narrow = a.fast && (long long)w < kDoubleExact / mult; // every cost an exact integer in a double
    // first layer a stage into v can start at
    for (int i = tid; i < W * M; i += blockDim.x) {
        const int v = i / M, d = i - v * M + 1;
        const unsigned long long room = (unsigned long long)a.cap > 0x7FFFFFFFFFFFFFFFull / d ? 0x7FFFFFFFFFFFFFFFull
                                                                                              : (unsigned long long)a.cap * d;
        int lo = s_lf[i], hi = v; // ceil(bytes / d) <= cap; nothing fits: v
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_pm[v] - s_pm[mid] <= room) hi = mid; else lo = mid + 1;
        }
        a.flo[i] = (unsigned char)lo;
        s_lf[i] = (unsigned char)lo; // (only this thread reads entry i before the barrier)
    }
    if (st == OOB_OK && narrow) { // the fastest stage is one of a single layer
        double least = kNone;
        for (int i = tid; i < L * M; i += blockDim.x) {
            const int l = i / M, d = i - l * M;
            const double t = s_pt[(l + 1) * M + d] - s_pt[l * M + d] + (l + 1 < L ? (double)bnd[l] : 0.0);
            if (t > 0) least = fmin(least, t);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) least = fmin(least, __shfl_xor(least, d, 64));
        if (lane == 0) atomicMin(&s_min, (unsigned long long)__double_as_longlong(least));
    }
    wg_sync();
    int total = 0;
    if (st == OOB_OK && narrow) { // list the possible slowest stages by time
        const int kmin = (int)(s_min >> 44);
        const unsigned inv = recip(M);
        for (int pass = 0; pass < 2; ++pass) {
            for (int v = 1 + wave; v <= L; v += nw) { // a wave takes the stages that end at layer v
                const double x = v < L ? (double)bnd[v - 1] : 0.0;
                for (int i0 = lane; i0 < v * M; i0 += 256) { // four entries of a lane in flight
                    double tau[4];
                    int pos[4], ud[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int i = i0 + 64 * q, ic = i < v * M ? i : 0;
                        const int u = quot(ic, inv), d = ic - u * M;
                        const bool ok = (i < v * M) & (u >= s_lf[v * M + d]);
                        tau[q] = s_pt[v * M + d] - s_pt[ic] + x;
                        ud[q] = u | (d + 1) << 16;
                        pos[q] = ok ? imax(0, imin((__double2hiint(tau[q]) >> 12) - kmin, kBins - 1)) : -1;
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) if (pos[q] >= 0) pos[q] = atomicAdd(&s_hist[pos[q]], 1);
                    if (pass)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (pos[q] >= 0) {
                                if (total <= room) s_list[pos[q]] = (unsigned)(ud[q] | v << 8);
                                else { a.ctau[pos[q]] = tau[q]; a.cuvd[pos[q]] = (unsigned)(ud[q] | v << 8); }
                            }
                }
            }
            wg_sync();
            if (pass) {
                // lists that fit are put in order in LDS and written out in a row
                if (total <= room)
                    for (int i = tid; i < total; i += blockDim.x) {
                        const unsigned uvd = s_list[i];
                        const int u = uvd & 255, v = uvd >> 8 & 255, d = (int)(uvd >> 16) - 1;
                        a.ctau[i] = s_pt[v * M + d] - s_pt[u * M + d] + (v < L ? (double)bnd[v - 1] : 0.0);
                        a.cuvd[i] = uvd;
                    }
                break;
            }
            // exclusive scan of the bins: kBins / kPrepThreads each
            constexpr int per = kBins / kPrepThreads;
            int h[per], sum = 0;
#pragma unroll
            for (int q = 0; q < per; ++q) { h[q] = s_hist[tid * per + q]; sum += h[q]; }
            int incl = sum;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) { const int y = __shfl_up(incl, d, 64); if (lane >= d) incl += y; }
            if (lane == 63) s_wave[wave] = incl;
            wg_sync();
            int base = incl - sum;
            for (int i = 0; i < nw; ++i) { if (i < wave) base += s_wave[i]; total += s_wave[i]; }
#pragma unroll
            for (int q = 0; q < per; ++q) { s_hist[tid * per + q] = base; base += h[q]; }
            wg_sync();
        }
    }
    if (tid == 0) {
        *a.status = st;
        Head h;
        h.ncand = (unsigned)total;
        h.bucket = (unsigned)imax(bucket_least(a.nk), (total + kMaxBuckets - 1) / kMaxBuckets);
        h.nbuckets = ((unsigned)total + h.bucket - 1) / h.bucket;
        h.alive = h.next = h.done = h.over = 0;
        h.narrow = narrow;
        *a.head = h;
    }
}

// ---------------------------------------------------------------------------------------------
// Shared pieces of the LDS kernels.
// ---------------------------------------------------------------------------------------------
// What one wave has written to LDS is read by its other lanes: program order of the LDS operations
// of a wave is execution order, the fences keep the compiler from moving them.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Minimum over aligned groups of 4 / 16 consecutive lanes, in every lane of the group, with data-parallel
// moves (quad permutations 1,0,3,2 and 2,3,0,1; then the mirror images within each half row and row,
// which hand every lane a lane of the other half).
template <int CTRL> __device__ __forceinline__ double dpp_f64(double x) {
    int lo = __double2loint(x), hi = __double2hiint(x);
    lo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false);
    hi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double min4(double x) {
    x = fmin(x, dpp_f64<0xB1>(x));
    return fmin(x, dpp_f64<0x4E>(x));
}
__device__ __forceinline__ double min16(double x) {
    x = min4(x);
    x = fmin(x, dpp_f64<0x141>(x));
    return fmin(x, dpp_f64<0x140>(x));
}

// Lane 15 of the row below in rows 1 and 3 (rows 0 and 2: unchanged).
__device__ __forceinline__ double row_below(double x) {
    int lo = __double2loint(x), hi = __double2hiint(x);
    lo = __builtin_amdgcn_update_dpp(lo, lo, 0x142, 0xA, 0xF, false);
    hi = __builtin_amdgcn_update_dpp(hi, hi, 0x142, 0xA, 0xF, false);
    return __hiloint2double(hi, lo);
}

// The profile in LDS: PT[l ms + d-1] prefix sums, PX = PT plus the boundary term of a stage ending at layer l,
// X the boundary terms, flo as in Args.  At eight GPUs per node a row is nine doubles where there is room (ms = M | 1, PAD): neighbouring
// lanes read neighbouring rows, which fall on the same few banks otherwise (47-63 % of the LDS cycles were conflicts): 98 layers 780 ->
// 662 us, 61 layers, 18 nodes 672 -> 660 us; 48 layers with the limit binding, in the bounds only: within what runs differ by.  SUM: PX is not kept but added up where it is read (integers below 2^52: the same
// value), for shapes whose tables leave it no room.
struct Prof { double *PT, *PX, *X; unsigned char *flo; };
template <bool SUM> __device__ __forceinline__ double stage_end(const Prof &s, int l, int i) { // i = l ms + d-1
    if constexpr (SUM) return s.PT[i] + s.X[l];
    else return s.PX[i];
}
template <bool SUM> __device__ __forceinline__ Prof load_prof(const Args &a, double *lds, int ms) {
    const int W = a.L + 1, n = W * a.M;
    Prof p;
    p.PT = lds; p.PX = p.PT + W * ms; p.X = SUM ? p.PX : p.PX + W * ms; p.flo = (unsigned char *)(p.X + W);
    const long long *bnd = (const long long *)a.prof.boundary_ns;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int l = i / a.M, at = ms == a.M ? i : l * ms + (i - l * a.M);
        const double pt = (double)a.PT[i];
        p.PT[at] = pt;
        if (!SUM) p.PX[at] = pt + (l > 0 && l < a.L ? (double)bnd[l - 1] : 0.0);
        p.flo[i] = a.flo[i];
    }
    for (int l = threadIdx.x; l < W; l += blockDim.x) p.X[l] = l > 0 && l < a.L ? (double)bnd[l - 1] : 0.0;
    return p;
}
// Whether the ends of stages that are not the model's last ascend with the layer on every number of GPUs, as far as this thread
// looks (the threads of the workgroup share the layers out).
template <bool PAD> __device__ __forceinline__ bool ends_ascend(const Prof &s, int L, int M) {
    bool up = true;
    for (int i = threadIdx.x; i < (L - 2) * M; i += blockDim.x) {
        const int at = (1 + i / M) * (PAD ? M | 1 : M) + i % M;
        up = up && s.PX[at] <= s.PX[at + (PAD ? M | 1 : M)];
    }
    return up;
}
// Reach of a stage on dd GPUs into layer p (before the slowest stage: it starts at r .. p-1; p: none) that
// takes less than tau (STRICT) or at most tau: it only gets slower and heavier as its start goes down.
template <bool STRICT, bool SUM>
__device__ __forceinline__ int reach_back(const Prof &s, int M, int ms, int p, int dd, double tau) {
    const double end = stage_end<SUM>(s, p, p * ms + dd - 1);
    int lo = s.flo[p * M + dd - 1], hi = p;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const double t = end - s.PT[mid * ms + dd - 1];
        if (STRICT ? t < tau : t <= tau) hi = mid; else lo = mid + 1;
    }
    return lo;
}
// Reach of a stage on dd GPUs out of layer p (after the slowest stage: it ends at p+1 .. r; p: none).  Impossible
// stays impossible and the time without the boundary term only grows as the end goes up.
__device__ __forceinline__ int reach_on(const Prof &s, int L, int M, int ms, int p, int dd, double tau) {
    const double start = s.PT[p * ms + dd - 1];
    int lo = p, hi = L;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s.flo[mid * M + dd - 1] <= p && s.PT[mid * ms + dd - 1] - start <= tau) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------------------------
// Lower bounds.  For a bucket of slowest stages with times lo .. hi and multipliers lambda (per GPU) and
// mu (per stage) the cost of any pipeline of n nodes around one of them is at least
//     mid tau + P[u] + S[v] + lambda d + mu - lambda n M - mu S_max,
// P[u] / S[v] = least sum over the stages of [0, u) / [v, L) of (weighted time + lambda GPUs + mu), stage times
// at most hi, tau's share in a weight taken from the end of the bucket that makes it smaller: exactly n M
// GPUs and at most S_max stages are used, whatever the prices.  The bound is the largest over the
// multipliers.  Row after row of the two paths.  With prices of stages, and where stages of more than kRing layers are
// fast enough: a wave takes two or four lambdas, thirty-two or sixteen lanes each share out the starts of the last stage, and the
// cost of a stage, which does not hang on mu, serves every mu of the wave; what hangs on the row alone is read once for the wave.  Else
// path_rows().  Bound by the chain of rows (LDS reads, the GPU counts one after the other, reduction over the lanes) at one
// workgroup per bucket: 120 us at 98 layers x 8 GPUs, 512 buckets, and 79 us at 48 layers with 64 pairs of multipliers (348 with
// a path per pair, the prices formed again for every entry and template at the end).  The ends of stages count with
// their boundary term (less so before: 2 400 instead of 2 000 evaluations at 98 layers).
// ---------------------------------------------------------------------------------------------
__device__ const double kLambdaGiven[kLambdas] = {0, 0.04, 0.1, 0.2, 0.4, 0.8, 1.6, 3.5}; // more nodes pay (C falls with n) ...
__device__ const double kLambda4S[kLambdas] = {0, -0.06, -0.14, -0.25, -0.43, -0.7, -1.3, -3.5}; // ... or cost
__device__ const double kMuStep[kMus] = {0, 0.1, 0.2, 0.35, 0.5, 0.75, 1, 1.5};

// Fewest nodes that can cover the layers at all with stages of at most the bucket's slowest time (boundary terms left
// out of the test, so never too many).  One wave, lane = start layer: the farthest layer that g GPUs of a node
// reach follows from the farthest that fewer do, because a stage that starts later also ends later; then node after
// node from the farthest layer so far.
constexpr int kCoverGpus = 8;
__device__ int fewest_nodes(int L, int M, const unsigned char *reach, unsigned char *s_far) {
    const int lane = threadIdx.x & 63;
    int before = 0; // farthest of the start layers before this round's
    for (int q0 = 0; q0 < L; q0 += 64) {
        const int q = imin(q0 + lane, L - 1);
        int far[kCoverGpus + 1];
        far[0] = q;
#pragma unroll
        for (int g = 1; g <= kCoverGpus; ++g) far[g] = q;
#pragma unroll
        for (int g = 0; g < kCoverGpus; ++g)
#pragma unroll
            for (int dd = 1; dd <= kCoverGpus - g; ++dd)
                if (g + dd <= M && far[g] < L) far[g + dd] = imax(far[g + dd], (int)reach[far[g] * M + dd - 1]);
                else if (g + dd <= M) far[g + dd] = L;
        int f = q;
#pragma unroll
        for (int g = 1; g <= kCoverGpus; ++g) if (g == M) f = far[g];
        f = imax(scan_max(f, lane), before);
        if (q0 + lane < L) s_far[q0 + lane] = (unsigned char)f;
        before = __shfl(f, 63, 64);
    }
    wave_sync();
    int n = 0, at = 0;
    while (at < L && n <= L) { // (a node that covers nothing: never)
        const int to = s_far[at];
        if (to <= at) return L + 1;
        at = to;
        ++n;
    }
    return n;
}

// What the multipliers k take off for a pipeline of n nodes, in units of the bucket's fastest stage.
__device__ __forceinline__ double spent(const Args &a, int k, int n) {
    return (a.Nb > 0 ? kLambdaGiven[k % kLambdas] : kLambda4S[k % kLambdas]) * (n * a.M) + kMuStep[k / kLambdas] * a.Smax;
}
// The bound of an entry (its values lb[0 .. nk-1]) of a bucket for n <= a.top nodes; below all doubt where there is none.
__device__ __forceinline__ double bound_of(const Args &a, const float *lb, double lo, int fewest, int n) {
    if (n < fewest) return kNone;
    double x = -kNone;
    for (int k = 0; k < a.nk; ++k) x = fmax(x, (double)lb[k] - lo * spent(a, k, n));
    return x;
}
// The rows of one side's path without prices of stages where no stage has more than K layers, one wave: lane = (lambda, GPU
// count).  A lane keeps, per layer x so far, the path up to x plus what x adds to the time of a stage on its GPUs, and takes
// the least over as many x as such a stage may have layers.  The last K of them are in LDS, no lane reads another's, and all
// but the newest two are read a row ahead.  One wave does for a side what four do with the starts shared out: 64 000 cycles
// instead of 90 000-130 000 for stages of up to 8 layers, 95 000 instead of 140 000 up to 16 (98 layers x 8 GPUs).
constexpr int kRing = 16;
template <int MT, bool PAD, bool SIDE, int K>
__device__ __forceinline__ void path_rows(const Prof &s, int L, const unsigned char *reach, double price, double extra, double *P, double *ring) {
    constexpr int M = MT, ms = PAD ? M | 1 : M;
    const int lane = threadIdx.x & 63, d = lane & (M - 1);
    const double *near = (SIDE ? s.PT : s.PX) + d, *far = (SIDE ? s.PX : s.PT) + d;
    const double sign = SIDE ? 2.0 : -1.0;
    double *const mine = ring + lane;
    double last = 0.0, g1 = kNone, old[K]; // the path up to the layer before; what the one before that adds, and those before it (k = 2 ..)
#pragma unroll
    for (int k = 2; k < K; ++k) old[k] = kNone;
    auto of = [=](int row) { return SIDE ? L - row : row; };
    int rc = reach[of(1) * M + d];
    double here = near[of(1) * ms], there = far[of(0) * ms];
    for (int row = 1; row <= L; ++row) {
        // stages [x, p) before, [p, x) after the slowest stage
        const int p = of(row), lim = SIDE ? rc - p : p - rc, pn = of(imin(row + 1, L));
        double acc = 1 < lim ? g1 : kNone;
#pragma unroll
        for (int k = 2; k < K; ++k) if (k < lim) acc = fmin(acc, old[k]);
        const double g0 = fma(sign, there, last), h = here;
        rc = reach[pn * M + d];
        here = near[pn * ms];
        there = far[p * ms];
        mine[(row & (kRing - 1)) * 64] = g1;
#pragma unroll
        for (int k = 2; k < K; ++k) old[k] = mine[((row + 2 - k) & (kRing - 1)) * 64]; // of the next row (before the first: not used)
        if (lim > 0) acc = fmin(acc, g0);
        g1 = g0;
        acc = fma(-sign, h, acc) + price;
        if (M >= 2) acc = fmin(acc, dpp_f64<0xB1>(acc));
        if (M >= 4) acc = fmin(acc, dpp_f64<0x4E>(acc));
        if (M >= 8) acc = fmin(acc, dpp_f64<0x141>(acc));
        last = acc + extra;
        if (d == 0 && lane < kLambdas * M) P[p] = last;
    }
    wave_sync();
}
// Five waves per SIMD asked for, two workgroups per compute unit; with prices of stages three: a workgroup has most of the LDS there.
template <int MT, bool PAD, bool MUS>
__global__ void __launch_bounds__(kBoundThreads, MUS ? 3 : 5) k_exact_bounds(Args a, int mus) {
    constexpr int CW = MT ? MT : 8, KL = MUS ? 16 : 32, LL = 64 / KL, MH = MUS ? kMus / 2 : 1; // lanes of a lambda, lambdas and mus of a wave
    HIP_DYNAMIC_SHARED(double, s_dyn)
    __shared__ unsigned long long s_lo, s_hi;
    __shared__ double s_lam[kLambdas], s_mu[kMus];
    __shared__ int s_fewest, s_up, s_most[2];
    if (*a.status != OOB_OK || !a.head->narrow) return;
    const unsigned b = blockIdx.x, K = a.head->bucket;
    if (b >= a.head->nbuckets) return;
    const int L = a.L, M = MT ? MT : a.M, W = L + 1, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned c0 = b * K, c1 = min(a.head->ncand, c0 + K);
    const int ms = PAD ? M | 1 : M;
    const Prof s = load_prof<false>(a, s_dyn, ms);
    unsigned char *rb = (unsigned char *)(s_dyn + prof_doubles(L, M, ms)), *rf = rb + ((size_t)W * M + 7) / 8 * 8;
    double *PS = (double *)(rf + ((size_t)W * M + 7) / 8 * 8); // [mu][lambda][side][L+1]
    float *s_lb = (float *)(PS + (size_t)mus * kLambdas * 2 * W); // [kBucket][kMaxCount]
    double *s_ring = (double *)s_lb;                              // [2][kRing][64] for path_rows(), before that
    unsigned char *s_far = (unsigned char *)(s_lb + kBucket * kMaxCount); // [256] for fewest_nodes()
    static_assert(2 * kRing * 64 * sizeof(double) <= kBucket * kMaxCount * sizeof(float), "");
    if (threadIdx.x == 0) { s_lo = kNoneBits; s_hi = 0; s_fewest = 0; s_up = 1; s_most[0] = s_most[1] = 0; }
    wg_sync();
    if (!ends_ascend<PAD>(s, L, M)) s_up = 0;
    for (unsigned c = c0 + threadIdx.x; c < c1; c += blockDim.x) {
        atomicMin(&s_lo, (unsigned long long)__double_as_longlong(a.ctau[c]));
        atomicMax(&s_hi, (unsigned long long)__double_as_longlong(a.ctau[c]));
    }
    wg_sync();
    const double lo = __longlong_as_double((long long)s_lo), hi = __longlong_as_double((long long)s_hi);
    int mostP = 0, mostS = 0; // layers of the longest stage
    for (int i = threadIdx.x; i < W * M; i += blockDim.x) {
        const int p = i / M, dd = i - p * M + 1;
        const int back = reach_back<false, false>(s, M, ms, p, dd, hi);
        rb[i] = (unsigned char)back;
        int on = reach_on(s, L, M, ms, p, dd, hi);
        // no end of a stage beyond this is fast enough (where they are, but for the model's end, ascending: else more are let through)
        if (on < L && s_up) while (on > p && s.PX[on * ms + dd - 1] - s.PT[p * ms + dd - 1] > hi) --on;
        rf[i] = (unsigned char)on;
        mostP = imax(mostP, p - back);
        mostS = imax(mostS, on - p);
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) { mostP = imax(mostP, __shfl_xor(mostP, m, 64)); mostS = imax(mostS, __shfl_xor(mostS, m, 64)); }
    if (lane == 0) { atomicMax(&s_most[0], mostP); atomicMax(&s_most[1], mostS); }
    const bool given = a.Nb > 0;
    if (threadIdx.x < kLambdas) s_lam[threadIdx.x] = (given ? kLambdaGiven[threadIdx.x] : kLambda4S[threadIdx.x]) * lo;
    else if (threadIdx.x - kLambdas < kMus) s_mu[threadIdx.x - kLambdas] = kMuStep[threadIdx.x - kLambdas] * lo;
    wg_sync();
    const double pw = given ? 0.0 : 4.0 * lo, sw = given ? -hi : 3.0 * lo, mid = given ? (double)a.Nb : 4.0;
    const int nt = nw - 1; // the last wave: fewest nodes
    if (wave == nt && M <= kCoverGpus) {
        const int n = fewest_nodes(L, M, rf, s_far);
        if (lane == 0) s_fewest = n;
    }
    bool done = false; // the rows, one wave a side
    if constexpr (MT != 0 && !MUS) {
        const int most = imax(s_most[0], s_most[1]), li = imin(lane / MT, kLambdas - 1);
        done = most <= kRing;
        if (done && wave < 2) {
            double *P = PS + ((size_t)li * 2 + wave) * W;
            const double price = s_lam[li] * (lane % MT + 1);
            if (lane % MT == 0 && lane < kLambdas * MT) P[wave ? L : 0] = 0.0;
            if (wave == 0) {
                if (most <= 8) path_rows<MT, PAD, false, 8>(s, L, rb, price, pw + s_mu[0], P, s_ring);
                else path_rows<MT, PAD, false, kRing>(s, L, rb, price, pw + s_mu[0], P, s_ring);
            } else {
                if (most <= 8) path_rows<MT, PAD, true, 8>(s, L, rf, price, sw + s_mu[0], P, s_ring + kRing * 64);
                else path_rows<MT, PAD, true, kRing>(s, L, rf, price, sw + s_mu[0], P, s_ring + kRing * 64);
            }
        }
    }
    if (!done) {
    const int kp = lane & (KL - 1), each = MUS ? (mus + 1) / 2 : 1; // mus of a task
    for (int task = wave; wave < nt && task < 2 * (kLambdas / LL) * (MUS ? 2 : 1); task += nt) { // one side
        const int side = task & 1, li = (task >> 1) % (kLambdas / LL) * LL + lane / KL, m0 = (task >> 1) / (kLambdas / LL) * each, mn = MUS ? imin(each, mus - m0) : 1;
        const double l = s_lam[li];
        double *P = PS + ((size_t)(m0 * kLambdas + li) * 2 + side) * W; // of the task's first mu
        const int next_mu = kLambdas * 2 * W;
        for (int i = 0; i < mn; ++i)
            for (int x = kp; x <= L; x += KL) P[i * next_mu + x] = x == (side ? L : 0) ? 0.0 : kNone;
        double ld[CW];
#pragma unroll
        for (int j = 0; j < CW; ++j) ld[j] = l * (j + 1);
        double extra[MH];
#pragma unroll
        for (int i = 0; i < MH; ++i) extra[i] = (side ? sw : pw) + s_mu[imin(m0 + i, kMus - 1)];
        wave_sync();
        auto rows = [&](auto side_c) {
        constexpr bool side = decltype(side_c)::value;
        const double *near = side ? s.PT : s.PX, *far = side ? s.PX : s.PT;
        const unsigned char *reach = side ? rf : rb;
        for (int row = 1; row <= L; ++row) {
            // stages [x, row) before, [p, x) after the slowest stage; what hangs on p alone is the same in all lanes
            const int p = side ? L - row : row;
            double acc[MH];
#pragma unroll
            for (int i = 0; i < MH; ++i) acc[i] = kNone;
            for (int d0 = 0; d0 < M; d0 += CW) {
                int lim[CW], most = 0; // layers of the longest stage per GPU count
                double e[CW];
#pragma unroll
                for (int j = 0; j < CW; ++j) {
                    const int dc = MT ? j : imin(d0 + j, M - 1), rc = __builtin_amdgcn_readfirstlane(reach[p * M + dc]);
                    e[j] = near[p * ms + dc];
                    lim[j] = d0 + j < M ? (side ? rc - p : p - rc) : 0;
                    most = imax(most, lim[j]);
                }
                const double shift = MT ? 0.0 : l * d0;
                for (int k0 = 0; k0 < most; k0 += KL) { // stages of k + 1 layers
                    const int k = k0 + kp, x = side ? imin(p + 1 + k, L) : imax(p - 1 - k, 0);
                    double f[CW], v = kNone;
#pragma unroll
                    for (int j = 0; j < CW; ++j) f[j] = far[x * ms + (MT ? j : imin(d0 + j, M - 1))];
                    double px[MH];
#pragma unroll
                    for (int i = 0; i < MH; ++i) if (i < mn) px[i] = P[i * next_mu + x];
#pragma unroll
                    for (int j = 0; j < CW; ++j) {
                        const double c = side ? fma(2.0, f[j] - e[j], ld[j]) : (e[j] - f[j]) + ld[j];
                        if (k < lim[j]) v = fmin(v, c);
                    }
                    if (!MT) v += shift;
#pragma unroll
                    for (int i = 0; i < MH; ++i) if (i < mn) acc[i] = fmin(acc[i], px[i] + v);
                }
            }
#pragma unroll
            for (int i = 0; i < MH; ++i)
                if (i < mn) {
                    double x = min16(acc[i]);
                    if (KL == 32) x = fmin(x, row_below(x)); // (the upper row of either half: the minimum of both)
                    if (kp == KL - 1) P[i * next_mu + p] = x + extra[i];
                }
            wave_sync();
        }
        };
        if (side) rows(std::true_type{}); else rows(std::false_type{});
    }
    }
    wg_sync();
    // Roundings: at most six per stage, so 6 L 2^-53 < 2e-13 of what is added up.  That is prices and stage times (a
    // path may use 255 times the GPUs of the pipeline: lowered by 1e-9 of them), and prefix sums of the GPU count in use,
    // twice over -- which hold also the layers whose time on that count no stage takes (by 1e-12 of the largest).
    double total = 0;
    for (int d = 0; d < M; ++d) total = fmax(total, s.PT[L * ms + d]);
    // bounds of the bucket's entries, kBucket at a time; the smallest of every template
    const int count = a.n_max - a.n_min + 1, nk = mus * kLambdas;
    int lg = 0; // lanes per entry: the templates, rounded up to a power of two
    while (1 << lg < a.live) ++lg;
    const int E = 64 >> lg, ni = lane & ((1 << lg) - 1), n = a.n_min + ni;
    double lam[kLambdas]; // what the prices of n nodes' GPUs take off
#pragma unroll
    for (int i = 0; i < kLambdas; ++i) lam[i] = s_lam[i] * (n * M);
    float mine = __builtin_huge_valf();
    unsigned arg = c0;
    for (unsigned m0 = c0; m0 < c1; m0 += kBucket) {
        const int m = (int)min(c1 - m0, (unsigned)kBucket);
        for (int i = threadIdx.x; i < m * nk; i += blockDim.x) {
            const int q = i / nk, k = i - q * nk;
            const unsigned uvd = a.cuvd[m0 + q];
            const int u = uvd & 255, v = uvd >> 8 & 255, d = uvd >> 16;
            const double tau = a.ctau[m0 + q], l = s_lam[k % kLambdas], mu = s_mu[k / kLambdas];
            const double base = mid * tau + PS[(size_t)k * 2 * W + u] + PS[((size_t)k * 2 + 1) * W + v] + l * d + mu;
            const double low = base - 1e-9 * (fabs(base) + mid * tau + fabs(l) * a.n_max * M + mu * a.Smax) - 1e-12 * total;
            // a side that stages of at most the bucket's slowest time cannot cover: no pipeline (and no infinity minus another)
            s_lb[i] = base < kNone ? __double2float_rd(low) : __builtin_huge_valf();
            a.lb[(size_t)m0 * nk + i] = s_lb[i];
        }
        wg_sync();
        // lanes: as many entries as have lanes for their templates; the entries shared out among the waves
        for (int q0 = wave * E; q0 < m; q0 += nw * E) {
            const int q = imin(q0 + (lane >> lg), m - 1);
            double x = -kNone;
            for (int mi = 0; mi < mus; ++mi) {
                const float2 *f = (const float2 *)(s_lb + (q * mus + mi) * kLambdas);
                double y = -kNone;
#pragma unroll
                for (int i = 0; i < kLambdas; i += 2) y = fmax(y, fmax((double)f[i / 2].x - lam[i], (double)f[i / 2].y - lam[i + 1]));
                x = fmax(x, y - s_mu[mi] * a.Smax);
            }
            if (n < s_fewest || ni >= a.live) x = kNone;
            if (x < (double)mine) { mine = __double2float_rd(x); arg = m0 + q; }
        }
        wg_sync();
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) // the entries side by side: smallest bound, then first entry
        if (d >= 1 << lg) {
            const float f = __shfl_xor(mine, d, 64);
            const unsigned g = (unsigned)__shfl_xor((int)arg, d, 64);
            if (f < mine || (f == mine && g < arg)) { mine = f; arg = g; }
        }
    // (count <= kMaxCount = 64: a lane of the first wave has one template; those beyond the live ones have no bound)
    s_lb[threadIdx.x] = mine;
    ((unsigned *)s_lb)[kBoundThreads + threadIdx.x] = arg;
    wg_sync();
    if ((int)threadIdx.x < count) {
        for (int w = 1; w < nw; ++w) {
            const float f = s_lb[w * 64 + threadIdx.x];
            if (f < mine) { mine = f; arg = ((unsigned *)s_lb)[kBoundThreads + w * 64 + threadIdx.x]; }
        }
        if ((int)threadIdx.x >= a.live) { mine = __builtin_huge_valf(); arg = c0; }
        a.blb[(size_t)b * count + threadIdx.x] = mine;
        a.barg[(size_t)b * count + threadIdx.x] = (unsigned short)(arg - c0);
    }
    if (threadIdx.x == 0) { a.blo[b] = lo; a.bfew[b] = s_fewest; }
}

// Entries whose bound does not exceed the minimum found so far for some template: one wave each.
__device__ __forceinline__ double best_now(const Args &a, int i) {
    return __longlong_as_double((long long)__hip_atomic_load(&a.best[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// A wave looks through kFilterEntries consecutive entries, as many at once as have lanes for their templates, and appends
// what is left with one atomic.  What the multipliers take off per template is formed once per workgroup.  Bound by the
// loads of the bounds (64 numbers an entry with eight mus): 388 -> 8 us for 48 layers x 8 GPUs with the stage
// limit binding, 52 -> 12 us at 98 layers x 8 GPUs, against one entry at a time and 64 entries a wave.
constexpr int kFilterEntries = 16, kFilterThreads = 256;
__global__ void __launch_bounds__(kFilterThreads) k_exact_filter(Args a) {
    HIP_DYNAMIC_SHARED(double, s_spent) // [nk][live]
    if (*a.status != OOB_OK || !a.head->narrow) return;
    const int lane = threadIdx.x & 63, live = a.live;
    const unsigned total = a.head->ncand, w0 = blockIdx.x * (kFilterThreads / 64) * kFilterEntries;
    if (w0 >= total) return;
    for (int i = threadIdx.x; i < a.nk * live; i += kFilterThreads) s_spent[i] = spent(a, i / live, a.n_min + i % live);
    wg_sync();
    const unsigned c0 = w0 + (threadIdx.x >> 6) * kFilterEntries;
    if (c0 >= total) return;
    int lg = 2; // lanes per entry: the templates, rounded up to a power of two
    while (1 << lg < live) ++lg;
    const int E = 64 >> lg, ni = lane & ((1 << lg) - 1);
    const double best = ni < live ? __longlong_as_double((long long)a.best[ni]) : -1.0;
    const unsigned long long group = lg == 6 ? ~0ull : (1ull << (1 << lg)) - 1;
    unsigned keep = 0;
    const unsigned K = a.head->bucket;
    for (int q0 = 0; q0 < kFilterEntries; q0 += E) {
        const int q = q0 + (lane >> lg);
        const unsigned c = c0 + q;
        bool in = q < kFilterEntries && c < total && ni < live;
        if (in) {
            const unsigned bk = c / K;
            const double lo = a.blo[bk];
            const float4 *lb = (const float4 *)(a.lb + (size_t)c * a.nk); // (nk is a multiple of eight)
            double x = -kNone;
            for (int k = 0; k < a.nk; k += 8) {
                const float4 f = lb[k / 4], g = lb[k / 4 + 1];
                const double *sp = s_spent + k * live + ni;
                x = fmax(fmax(x, (double)f.x - lo * sp[0]), fmax((double)f.y - lo * sp[live], (double)f.z - lo * sp[2 * live]));
                x = fmax(fmax(x, (double)f.w - lo * sp[3 * live]), fmax((double)g.x - lo * sp[4 * live], (double)g.y - lo * sp[5 * live]));
                x = fmax(x, fmax((double)g.z - lo * sp[6 * live], (double)g.w - lo * sp[7 * live]));
            }
            in = a.n_min + ni >= a.bfew[bk] && x < kNone && x <= best;
        }
        const unsigned long long m = __ballot(in);
        for (int e = 0; e < E && q0 + e < kFilterEntries; ++e)
            if (m >> (e << lg) & group) keep |= 1u << (q0 + e);
    }
    unsigned at = 0;
    if (lane == 0 && keep) at = atomicAdd(&a.head->alive, (unsigned)__popc(keep));
    at = __shfl(at, 0, 64);
    if (lane < kFilterEntries && keep >> lane & 1) a.list[at + __popc(keep & ((1u << lane) - 1))] = c0 + lane;
}

// ---------------------------------------------------------------------------------------------
// Exact evaluation.  Bound by the steps of an entry, one after the other: at 98 layers x 8 GPUs the one-node tables are 60 % of its
// 69 000 cycles and the chain of nodes 25 %; the vector instructions of a launch are 47 us of its 104, two thirds of the wave cycles are waits, LDS and
// memory are far from busy.  81 us for the first picks and 124-130 us for the rest there
// (140-160 and 280-420 with the tables row after row in LDS; a version without a band,
// evaluating everything: 20.3 ms, 1.16 us per slowest stage).  J = number of stage counts kept per table
// entry: 1, or S_max + 1 (STAGED).
// ---------------------------------------------------------------------------------------------
struct Eval {
    Prof pr;
    unsigned char *reach; // [(L+1) M] of a stage into a layer p <= u / out of a layer p >= v
    double *pool;         // GU, W, then the waves' one-node tables
    unsigned pool_n;      // (sizes of tables are unsigned 32-bit numbers: signed ones cost k_exact_eval<false, 8> 16 more spilled registers, 64 bits 6)
    double *GU;           // [two sides][band][M, or staged_row(M)] covers next to the slowest stage, by the distance covered
    double *NP;           // [2 buffers][len+1 of both sides][J]
    double *OUT;          // [two sides][nodes][M][J] a whole nodes and g more GPUs
    int *ints;            // [0..1] bands
};
// Column of (g GPUs, j stages), 1 <= j <= g, in a row of a table with stage counts; column 0: impossible.
__host__ __device__ inline int staged_col(int g, int j) { return g * (g - 1) / 2 + j; }
__host__ __device__ inline int staged_row(int M) { return M * (M + 1) / 2 + 1; }
// Entry (r, j) of a band matrix with rows r = 1 .. and columns 0 .. len - r.
__device__ __forceinline__ int band_index(int r, int j, int len) { return (r - 1) * len - (r - 1) * (r - 2) / 2 + j; }
// One-node tables of a side (this wave's share): start positions idx = first .. in side coordinates (layers
// from the far end of the side), rows r = layers covered.  Lanes = (start, part of the walk, GPUs g); with stage
// counts the lanes that would share a walk out hold the counts j = 1 .. M instead.  A row takes the stages that
// cover its last k + 1 layers on CW GPU counts side by side: the CW table entries and the CW prefix sums of a
// step are read before any of them is used.
template <bool MIRROR, bool STAGED, int MT, bool SUM, bool PAD>
__device__ void one_node_tables(const Args &a, const Eval &e, int len, int band, double tau, double wt, double add,
                                double *Wm, double *GU, double *G, int first, int slots, int lgxs, int gbits) {
    constexpr int CW = MT ? MT : 8;
    const int L = a.L, M = MT ? MT : a.M, lane = threadIdx.x & 63;
    const int gi = lane & ((1 << gbits) - 1), xs = (lane >> gbits) & ((1 << lgxs) - 1), slot = lane >> (gbits + lgxs);
    const int idx = first + slot;
    const bool live = idx < len && slot < slots && gi < M;
    const int j = STAGED ? xs + 1 : 1;
    const int XS = STAGED ? 1 : 1 << lgxs, x0 = STAGED ? 0 : xs;
    const int row_n = STAGED ? staged_row(M) : M + 1;               // entries per row of a table
    double *T = G + (size_t)(slot < slots ? slot : 0) * (band + 1) * row_n; // (lanes beyond the tables read one and use nothing of it)
    const int g = gi + 1, rows = live ? imin(band, len - idx) : 0;
    const bool use = live && (!STAGED || j <= g);                   // this lane has an entry in every row
    const int q = live ? (MIRROR ? L - idx : idx) : 0;                           // start layer
    const int ms = PAD ? M | 1 : M;
    auto far = [&](int l, int gc) { return MIRROR ? stage_end<SUM>(e.pr, l, l * ms + gc) : e.pr.PT[l * ms + gc]; };
    const int top = g + 1 - (j - 1);
    const int none = 0; // row 0 holds no cover (a node's first stage is taken on its own): always impossible
    if (slot < slots && gi == 0 && xs == 0) T[none] = kNone;
    wave_sync();
    for (int r = 1; r <= band; ++r) {
        double acc = kNone;
        const bool on = use && r <= rows;
        const int p = on ? (MIRROR ? q - r : q + r) : 0;
        { // one stage on all g GPUs covers everything
            const int gc = imin(gi, M - 1), rc = e.reach[p * M + gc];
            const double here = MIRROR ? e.pr.PT[p * ms + gc] : stage_end<SUM>(e.pr, p, p * ms + gc), all = far(q, gc);
            const double tw = MIRROR ? all - here : here - all;
            const bool one = on & (j == 1) & (x0 == 0) & ((MIRROR ? rc - p : p - rc) >= r) & (!MIRROR | (tw <= tau));
            acc = one ? wt * tw + add : kNone;
        }
        for (int d0 = 0; d0 < M; d0 += CW) {
            double near[CW], late[CW]; // weighted share of layer p, latest end fast enough with its boundary term
            int lim[CW], off[CW]; // layers of the longest stage (the first layer of the node excluded), table column
            int most = 0;
#pragma unroll
            for (int w = 0; w < CW; ++w) {
                const int dc = MT ? w : imin(d0 + w, M - 1), rc = e.reach[p * M + dc];
                near[w] = wt * (MIRROR ? -e.pr.PT[p * ms + dc] : stage_end<SUM>(e.pr, p, p * ms + dc)) + add;
                late[w] = MIRROR ? e.pr.PT[p * ms + dc] + tau : 0.0;
                lim[w] = on && d0 + w + 1 < top ? imin(MIRROR ? rc - p : p - rc, r - 1) : 0; // the other stages need a GPU each
                most = imax(most, lim[w]);
                const int left = g - dc - 1; // GPUs of the other stages
                off[w] = (r - 1) * row_n + (STAGED ? (left > 0 && j > 1 ? staged_col(left, j - 1) : 0) : imax(left, 0));
            }
            for (int k = x0; __any(k < most); k += XS) { // stages of k + 1 layers
                const int kk = imin(k, imax(most - 1, 0)), x = on ? (MIRROR ? p + 1 + kk : p - 1 - kk) : 0;
                double tv[CW], gv[CW];
#pragma unroll
                for (int w = 0; w < CW; ++w) {
                    tv[w] = far(x, MT ? w : imin(d0 + w, M - 1));
                    gv[w] = T[k < lim[w] ? off[w] - kk * row_n : none]; // beyond the reach: an entry that is impossible
                }
#pragma unroll
                for (int w = 0; w < CW; ++w) {
                    const double c = gv[w] + (MIRROR ? fma(2.0, tv[w], near[w]) : near[w] - tv[w]); // (the weight is 2 after, 1 before)
                    acc = fmin(acc, (!MIRROR | (tv[w] <= late[w])) ? c : kNone);
                }
            }
        }
        if (!STAGED)
            for (int m = 1 << gbits; m < 1 << (gbits + lgxs); m <<= 1) acc = fmin(acc, __shfl_xor(acc, m, 64));
        if (on && (STAGED || xs == 0)) { // (entry 0 of a row, no GPU used: impossible)
            if (STAGED) {
                double *row = T + (size_t)r * row_n;
                row[staged_col(g, j)] = acc;
                if (g == 1) row[0] = kNone;
                if (g == M) Wm[(size_t)band_index(r, idx, len) * M + j - 1] = acc;
                if (idx + r == len) GU[(size_t)(r - 1) * row_n + staged_col(g, j)] = acc;
            } else {
                T[r * row_n + g] = acc;
                if (gi == 0) T[r * row_n] = kNone;
                if (g == M) Wm[band_index(r, idx, len)] = acc;
                else if (idx + r == len) GU[(r - 1) * M + g] = acc;
            }
        }
        wave_sync();
    }
}

// The value of the lane below (lane 0: its own), over the whole wave.
__device__ __forceinline__ double lane_below(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xF, 0xF, false), __builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xF, 0xF, false));
}
// The same tables in registers, for 1, 2, 4 or 8 GPUs per node and bands of up to 64 layers: a lane holds row r of a start (all g, with
// stage counts all j <= g), 64 / band starts side by side.  A cover on g' GPUs whose first layers a stage on d GPUs
// takes makes one on g' + d: g' goes up, and every row of it is final before it is used, so what depends on what is M
// steps long and not `band` rows.  The time of a stage is a difference of two prefix sums: the lane of the shorter
// cover adds its share, the wave hands the sum up a lane per layer of the stage, and the lane that wants it takes the
// minimum over as many as the stage may have layers (never past the first row of its own start).
// No LDS but the results: with stage counts the tables in LDS left room for two or three of sixteen waves.  Cycles of an entry in
// this phase, row after row in LDS and now: 98 layers x 8 GPUs 113 000 and 42 000 (call 711 -> 463 us), 48 layers with stage
// counts 730 000 and 141 000 (3.35 -> 1.10 ms), 26 layers x 4 GPUs 19 000 and 7 000.
template <bool MIRROR, bool STAGED, int MT, bool PAD>
__device__ __forceinline__ void node_tables(const Args &a, const Eval &e, int len, int band, double tau, double wt, double add, double *Wm, double *GU, int first, int slots) {
    constexpr int M = MT, J = STAGED ? M : 1;
    const int L = a.L, lane = threadIdx.x & 63, ms = PAD ? M | 1 : M;
    const int slot = lane / band, r = lane - slot * band + 1, idx = first + slot;
    const bool on = slot < slots && idx + r <= len;
    const int q = MIRROR ? L - idx : idx, p = on ? (MIRROR ? q - r : q + r) : 0;
    const double *here = (MIRROR ? e.pr.PT : e.pr.PX) + p * ms, *from = (MIRROR ? e.pr.PX : e.pr.PT) + p * ms; // as the end that a stage adds, as the one it starts from
    double T[M + 1][J + 1]; // [g][j], j = 1 without stage counts
    int lim[M];             // layers of the longest stage on d + 1 GPUs that leaves a layer to the others
#pragma unroll
    for (int d = 0; d < M; ++d) {
        const int rc = e.reach[p * M + d], n = MIRROR ? rc - p : p - rc;
        const double tw = MIRROR ? e.pr.PX[(on ? q : 0) * ms + d] - here[d] : here[d] - e.pr.PT[(on ? q : 0) * ms + d];
#pragma unroll
        for (int j = 1; j <= J; ++j) T[d + 1][j] = kNone;
        if (on & (n >= r) & (!MIRROR | (tw <= tau))) T[d + 1][1] = fma(wt, tw, add); // one stage on all of them
        lim[d] = on ? imin(n, r - 1) : 0;
    }
    if (MIRROR) // (the ends of the stages ascend: where the longest is not too slow with its boundary term, no shorter one is)
        for (bool more = true; __any(more);) {
            more = false;
#pragma unroll
            for (int d = 0; d < M; ++d) {
                const bool slow = lim[d] > 0 && e.pr.PX[(p + lim[d]) * ms + d] - here[d] > tau;
                lim[d] -= slow;
                more = more || slow;
            }
        }
#pragma unroll
    for (int g = 1; g < M; ++g)
#pragma unroll
        for (int d = 0; d + 1 + g <= M; ++d) {
            const double share = MIRROR ? wt * from[d] : -from[d], rest = (MIRROR ? -wt * here[d] : here[d]) + add;
            double h[J + 1], acc[J + 1];
#pragma unroll
            for (int j = 1; j <= J; ++j) if (j <= g) { h[j] = T[g][j] + share; acc[j] = kNone; }
            for (int k = 0; __any(k < lim[d]); ++k) {
#pragma unroll
                for (int j = 1; j <= J; ++j) if (j <= g) h[j] = lane_below(h[j]);
                if (k < lim[d])
#pragma unroll
                    for (int j = 1; j <= J; ++j) if (j <= g) acc[j] = fmin(acc[j], h[j]);
            }
#pragma unroll
            for (int j = 1; j <= J; ++j)
                if (j <= g) {
                    double &t = T[g + d + 1][STAGED ? imin(j + 1, J) : 1]; // (j <= g < M)
                    t = fmin(t, acc[j] + rest);
                }
        }
    if (!on) return;
#pragma unroll
    for (int j = 1; j <= J; ++j) Wm[(size_t)band_index(r, idx, len) * J + j - 1] = T[M][j];
    if (idx + r == len)
#pragma unroll
        for (int g = 1; g <= M; ++g)
#pragma unroll
            for (int j = 1; j <= J; ++j) {
                if (STAGED) { if (j <= g) GU[(r - 1) * staged_row(M) + staged_col(g, j)] = T[g][j]; }
                else if (g < M) GU[(r - 1) * M + g] = T[g][1];
            }
}

// c -> c + 1 whole nodes: nxt[p] = min over r of cur[p - r] + W[r][p - r] for this side, by nth threads (whole waves).
__device__ void node_step(int len, int band, int c, const double *Wm, const double *cur, double *nxt, int th, int nth) {
    const int lo = c + 1, hi = imin(len, (c + 1) * band), np = hi - lo + 1, h4 = th & 3;
    for (int i = th; i < ((np * 4 + 63) & ~63); i += nth) { // whole waves, four threads per position
        const int p = lo + (i >> 2), most = imin(band, p - c); // c nodes cover at least c layers
        double m = kNone;
        if (p <= hi)
            for (int r = 1 + h4; r <= most; r += 4) m = fmin(m, cur[p - r] + Wm[band_index(r, p - r, len)]);
        m = min4(m);
        if (h4 == 0 && p <= hi) nxt[p] = m;
    }
}
// OUT[c][g]: c whole nodes and g more GPUs next to the slowest stage cover the side.
__device__ void node_out(int M, int len, int band, int c, const double *cur, const double *GU, double *OUT, int th, int nth) {
    const int from = imax(1, len - c * band), to = imin(band, len - c); // distances left for the last node
    const bool whole = len >= c && len <= c * band;
    for (int i = th; i < ((M * 4 + 63) & ~63); i += nth) { // four threads per g
        const int g = i >> 2, h4 = i & 3;
        double m = kNone;
        if (g == 0) { if (h4 == 0 && whole) m = cur[len]; }
        else if (g < M) for (int r = from + h4; r <= to; r += 4) m = fmin(m, cur[len - r] + GU[(r - 1) * M + g]);
        m = min4(m);
        if (h4 == 0 && g < M) OUT[c * M + g] = m;
    }
}

// The same with stage counts: a thread takes kCounts neighbouring counts s of a cover by r layers and j stages more, so that of
// what it reads -- the M entries of the last node, the counts s - M .. s + kCounts - 2 of the cover before it -- each serves
// several sums (one count a thread, every sum two reads: 217 000 cycles an entry at 48 layers, 8 GPUs,
// 8 nodes; 80 000 now, with the waves of a side without layers put to the other's work; call 0.85 -> 0.56 ms).
// No count is below that of the nodes, so entry 0 of a row is impossible from one node on and stands for the counts below 0.
constexpr int kCounts = 4;
template <int MT>
__device__ __forceinline__ void add_node(const double *before, const double *node, int M, int s0, double *m) {
    constexpr int JM = MT ? MT : 8;
    double w[JM], x[JM + kCounts - 1];
#pragma unroll
    for (int j = 0; j < JM; ++j) w[j] = MT || j < M ? node[j] : kNone;
#pragma unroll
    for (int i = 0; i < JM + kCounts - 1; ++i) x[i] = before[imax(s0 - JM + i, 0)];
#pragma unroll
    for (int i = 0; i < kCounts; ++i)
#pragma unroll
        for (int j = 1; j <= JM; ++j) m[i] = fmin(m[i], x[JM + i - j] + w[j - 1]);
}
template <int MT>
__device__ void node_step_staged(const Args &a, int len, int band, int c, const double *Wm, const double *cur, double *nxt, int th, int nth) {
    const int J = a.Smax + 1, M = MT ? MT : a.M, lo = c + 1, hi = imin(len, (c + 1) * band), np = hi - lo + 1;
    if (c == 0) { // a single node
        for (int i = th; i < np * J; i += nth) {
            const int p = 1 + i / J, s = i % J;
            nxt[p * J + s] = s >= 1 && s <= M ? Wm[(size_t)band_index(p, 0, len) * M + s - 1] : kNone;
        }
        return;
    }
    const int groups = (J + kCounts - 1) / kCounts, items = np * groups, h4 = th & 3;
    for (int i = th; i < ((items * 4 + 63) & ~63); i += nth) { // whole waves, four threads per item
        const int it = imin(i >> 2, items - 1), p = lo + it / groups, s0 = it % groups * kCounts;
        const int least = imax(1, p - c * band), most = imin(band, p - c); // c nodes cover c layers at least and c band at most
        double m[kCounts];
#pragma unroll
        for (int q = 0; q < kCounts; ++q) m[q] = kNone;
        for (int r = least + h4; r <= most; r += 4) add_node<MT>(cur + (p - r) * J, Wm + (size_t)band_index(r, p - r, len) * M, M, s0, m);
#pragma unroll
        for (int q = 0; q < kCounts; ++q) {
            m[q] = min4(m[q]);
            if (h4 == q && i >> 2 < items && s0 + q < J) nxt[p * J + s0 + q] = m[q];
        }
    }
}
template <int MT>
__device__ void node_out_staged(const Args &a, int len, int band, int c, const double *cur, const double *GU, double *OUT, int th, int nth) {
    const int J = a.Smax + 1, M = MT ? MT : a.M, row_n = staged_row(M);
    const int from = imax(1, len - c * band), to = imin(band, len - c); // distances left for the last node
    double *const out = OUT + (size_t)c * M * J;
    if (c == 0) { // (a side of no layers: nothing is a cover)
        for (int i = th; i < M * J; i += nth) {
            const int g = i / J, s = i % J;
            out[i] = len == 0 ? (i == 0 ? 0.0 : kNone) : s >= 1 && s <= g && len <= band ? GU[(size_t)(len - 1) * row_n + staged_col(g, s)] : kNone;
        }
        return;
    }
    const bool whole = len >= c && len <= c * band;
    for (int s = th; s < J; s += nth) out[s] = whole ? cur[(size_t)len * J + s] : kNone; // g = 0
    const int groups = (J + kCounts - 1) / kCounts, items = (M - 1) * groups, h = th & 15;
    for (int i = th; i < ((items * 16 + 63) & ~63); i += nth) { // sixteen threads per item
        const int it = imin(i >> 4, items - 1), g = 1 + it / groups, s0 = it % groups * kCounts;
        double m[kCounts];
#pragma unroll
        for (int q = 0; q < kCounts; ++q) m[q] = kNone;
        for (int r = from + h; r <= to; r += 16) {
            const double *before = cur + (size_t)(len - r) * J, *node = GU + (size_t)(r - 1) * row_n + staged_col(g, 1);
            for (int j = 1; j <= g; ++j)
#pragma unroll
                for (int q = 0; q < kCounts; ++q) m[q] = fmin(m[q], before[imax(s0 + q - j, 0)] + node[j - 1]);
        }
#pragma unroll
        for (int q = 0; q < kCounts; ++q) {
            m[q] = min16(m[q]);
            if (h == q && i >> 4 < items && s0 + q < J) out[g * J + s0 + q] = m[q];
        }
    }
}

// The node-level recurrence of one side by one wave, in registers: lane p (and p + 64) holds NP_c[p] and the
// column W[1 .. B][p - r] it adds to; the wave shifts NP by a lane per r.  HIST[c][r] = NP_c[len - r], r = 0 .. band, is
// what the last node's partial covers need.  No LDS read and no barrier on the chain of up to n_max steps.
template <int B, bool TWO>
__device__ __forceinline__ void node_chain(int len, int band, int cend, const double *Wm, double *HIST) {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane)); // (or the places of W are formed once for all variants and kept in scratch memory: 5 000 cycles)
    double w0[B], w1[TWO ? B : 1];
    int at = lane - 1; // of W[r][lane - r]
#pragma unroll
    for (int r = 1; r <= B; ++r) {
        const bool in0 = (r <= band) & (lane >= r) & (lane <= len), in1 = (r <= band) & (lane + 64 <= len);
        w0[r - 1] = Wm[in0 ? at : 0];
        if (!in0) w0[r - 1] = kNone;
        if (TWO) {
            w1[r - 1] = Wm[in1 ? at + 64 : 0];
            if (!in1) w1[r - 1] = kNone;
        }
        at += len - r;
    }
    double c0 = lane == 0 ? 0.0 : kNone, c1 = kNone;
    for (int c = 0; c < cend; ++c) {
        if (lane <= len && len - lane <= band) HIST[c * (band + 1) + len - lane] = c0;
        if (TWO && lane + 64 <= len && len - lane - 64 <= band) HIST[c * (band + 1) + len - lane - 64] = c1;
        double n0 = kNone, n1 = kNone, s0 = c0, s1 = c1;
#pragma unroll
        for (int r = 1; r <= B; ++r) {
            if (TWO) { // lane 0 of the upper half takes the lower half's last
                int lo = __builtin_amdgcn_update_dpp(0, __double2loint(s0), 0x13C, 0xF, 0xF, false);
                int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(s0), 0x13C, 0xF, 0xF, false);
                s0 = __hiloint2double(lane == 0 ? 0x7FF00000 : hi, lane == 0 ? 0 : lo);
                lo = __builtin_amdgcn_update_dpp(lo, __double2loint(s1), 0x138, 0xF, 0xF, false);
                hi = __builtin_amdgcn_update_dpp(hi, __double2hiint(s1), 0x138, 0xF, 0xF, false);
                s1 = __hiloint2double(hi, lo);
                n1 = fmin(n1, s1 + w1[r - 1]);
            } else {
                const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(s0), 0x138, 0xF, 0xF, false);
                const int hi = __builtin_amdgcn_update_dpp(0x7FF00000, __double2hiint(s0), 0x138, 0xF, 0xF, false);
                s0 = __hiloint2double(hi, lo);
            }
            n0 = fmin(n0, s0 + w0[r - 1]);
        }
        c0 = n0;
        c1 = n1;
    }
}
constexpr int kChainBand = 16, kChainLen = 127;
__device__ __forceinline__ void node_chain_any(int len, int band, int cend, const double *Wm, double *HIST) {
    if (len < 64) {
        if (band <= 4) node_chain<4, false>(len, band, cend, Wm, HIST);
        else if (band <= 8) node_chain<8, false>(len, band, cend, Wm, HIST);
        else if (band <= 12) node_chain<12, false>(len, band, cend, Wm, HIST);
        else node_chain<kChainBand, false>(len, band, cend, Wm, HIST);
    } else {
        if (band <= 8) node_chain<8, true>(len, band, cend, Wm, HIST);
        else if (band <= 12) node_chain<12, true>(len, band, cend, Wm, HIST);
        else node_chain<kChainBand, true>(len, band, cend, Wm, HIST);
    }
}

// The slowest stage at every place it fits: ca whole nodes and g GPUs before it, cb whole nodes and M - d - g
// GPUs after it, n = ca + cb + 1, for every template up to nhi <= a.top.
template <bool STAGED>
__device__ void combine(const Args &a, const Eval &e, int d, double tau, int nhi, int cendP, int cendS, double mid,
                        unsigned long long *s_best) {
    const int L = a.L, M = a.M, J = STAGED ? a.Smax + 1 : 1;
    const int places = M - d + 1;
    for (int i = threadIdx.x; i < cendP * cendS; i += blockDim.x) {
        const int ca = i / cendS, cb = i - ca * cendS, n = ca + cb + 1;
        if (n < a.n_min || n > nhi) continue;
        double m = kNone;
        for (int g = 0; g < places; ++g) {
            if (!STAGED) m = fmin(m, e.OUT[ca * M + g] + e.OUT[(a.nodes + cb) * M + (M - d - g)]);
            else {
                const double *p = e.OUT + (size_t)(ca * M + g) * J, *s = e.OUT + (size_t)((a.nodes + cb) * M + (M - d - g)) * J;
                double pre = kNone; // least over the stages before, as many as the stages after leave room for
                int j1 = 0;
                for (int j2 = a.Smax - 1; j2 >= 0; --j2) {
                    for (; j1 + 1 + j2 <= a.Smax; ++j1) pre = fmin(pre, p[j1]);
                    m = fmin(m, pre + s[j2] - (double)j2 * tau);
                }
            }
        }
        m += mid * tau;
        if (m < kNone) atomicMin(&s_best[n - a.n_min], (unsigned long long)__double_as_longlong(m));
    }
}

// One row of the tables over (layers covered, GPUs used[, stages]) of a side: T[r][D][j], r layers from the far end of the
// side on D GPUs, node after node.  Called by nth threads (whole waves); a thread has one (D, j) and a share of the walk.
template <bool MIRROR, bool STAGED, int MT, bool SUM, bool PAD>
__device__ void gpu_row(const Args &a, const Eval &e, int r, int nd, int jd, double tau, double wt, double add, double *T, int th,
                        int nth) {
    constexpr int CW = MT ? MT : 8;
    const int L = a.L, M = MT ? MT : a.M, row_n = nd * jd, p = MIRROR ? L - r : r;
    const int items = STAGED ? nd * (jd - 1) : nd; // D = 0 .. nd - 1 (D = 0 covers nothing), j = 1 .. jd - 1
    int lg = 0;
    while (lg < 6 && items << (lg + 1) <= nth) ++lg;
    const int XS = 1 << lg, x0 = th & (XS - 1);
    const int ms = PAD ? M | 1 : M;
    auto far = [&](int l, int gc) { return MIRROR ? stage_end<SUM>(e.pr, l, l * ms + gc) : e.pr.PT[l * ms + gc]; };
    for (int i0 = 0; i0 < items; i0 += nth >> lg) {
        const int i = i0 + (th >> lg), D = i % nd, j = STAGED ? i / nd + 1 : 1;
        const bool on = i < items && D > 0 && j <= D;
        const int gD = on ? (D - 1) % M + 1 : 0; // GPUs of D's last node
        double acc = kNone;
        for (int d0 = 0; d0 < M; d0 += CW) {
            double near[CW];
            int lim[CW], off[CW], most = 0;
#pragma unroll
            for (int w = 0; w < CW; ++w) {
                const int dc = MT ? w : imin(d0 + w, M - 1), rc = e.reach[p * M + dc];
                near[w] = MIRROR ? e.pr.PT[p * ms + dc] : stage_end<SUM>(e.pr, p, p * ms + dc);
                lim[w] = d0 + w < gD && (!STAGED || D - dc - 1 >= j - 1) ? imin(MIRROR ? rc - p : p - rc, r) : 0;
                most = imax(most, lim[w]);
                off[w] = (r - 1) * row_n + imax(D - dc - 1, 0) * jd + (STAGED ? j - 1 : 0);
            }
            for (int k = x0; __any(k < most); k += XS) { // stages of k + 1 layers
                const int kk = imin(k, imax(most - 1, 0)), x = MIRROR ? p + 1 + kk : p - 1 - kk;
                double tv[CW], gv[CW];
#pragma unroll
                for (int w = 0; w < CW; ++w) {
                    tv[w] = far(x, MT ? w : imin(d0 + w, M - 1));
                    gv[w] = T[off[w] - kk * row_n];
                }
#pragma unroll
                for (int w = 0; w < CW; ++w) {
                    const double t = MIRROR ? tv[w] - near[w] : near[w] - tv[w];
                    const bool ok = (k < lim[w]) & (!MIRROR | (t <= tau));
                    const double c = gv[w] + (wt * t + add);
                    acc = fmin(acc, ok ? c : kNone);
                }
            }
        }
        for (int m = 1; m < XS; m <<= 1) acc = fmin(acc, __shfl_xor(acc, m, 64));
        if (x0 == 0 && i < items) {
            T[(size_t)r * row_n + D * jd + (STAGED ? j : 0)] = acc;
            if (STAGED && j == 1) T[(size_t)r * row_n + D * jd] = kNone;
        }
    }
}

// The cost of the best pipelines around slowest stage (u, v, d) with n <= nhi nodes, merged into s_best.
// Returns false (the same in every thread) if the tables do not fit the workgroup's LDS (STAGED only).
template <bool STAGED, int MT, bool SUM, bool PAD, bool REGS>
__device__ bool evaluate(const Args &a, Eval &e, unsigned uvd, double tau, int nhi, unsigned long long *s_best) {
    const int L = a.L, M = MT ? MT : a.M, J = STAGED ? a.Smax + 1 : 1, nw = blockDim.x >> 6, W = L + 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int u = uvd & 255, v = uvd >> 8 & 255, d = uvd >> 16;
    const int lenP = u, lenS = L - v;
    // ---- reach of the stages, and the most layers a node can cover on either side: a stage on dd GPUs covers at
    // most rho dd layers, rho the largest (layers / GPUs) of any stage, so a node at most floor(M rho)
    if (threadIdx.x < 2) e.ints[threadIdx.x] = 0;
    wg_sync();
    int mostP = 0, mostS = 0;
    const unsigned inv = recip(M);
    for (int i = threadIdx.x; i < W * M; i += blockDim.x) {
        const int p = quot(i, inv), dd = i - p * M + 1;
        int r = p;
        if (p >= 1 && p <= u) { r = reach_back<true, SUM>(e.pr, M, PAD ? M | 1 : M, p, dd, tau); mostP = imax(mostP, (p - r) * M / dd); }
        else if (p >= v && p < L) { r = reach_on(e.pr, L, M, PAD ? M | 1 : M, p, dd, tau); mostS = imax(mostS, (r - p) * M / dd); }
        e.reach[i] = (unsigned char)r;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) { mostP = imax(mostP, __shfl_xor(mostP, m, 64)); mostS = imax(mostS, __shfl_xor(mostS, m, 64)); }
    if ((threadIdx.x & 63) == 0) { atomicMax(&e.ints[0], mostP); atomicMax(&e.ints[1], mostS); }
    wg_sync();
    const int bandP = imin(e.ints[0], lenP), bandS = imin(e.ints[1], lenS);
    wg_sync();
    if ((lenP && !bandP) || (lenS && !bandS)) return true; // some layer fits no stage fast enough
    const double mid = a.Nb > 0 ? (double)a.Nb : 4.0;
    const double ptau = STAGED || a.Nb > 0 ? 0.0 : 4.0, stau = STAGED ? 0.0 : a.Nb > 0 ? -1.0 : 3.0;
    const int cendP = imin(nhi, lenP + 1), cendS = imin(nhi, lenS + 1); // a node covers at least one layer
    const int nwp = (nw + 1) >> 1, mir = wave >= nwp; // half of the waves per side
    const int th = mir ? (int)threadIdx.x - nwp * 64 : (int)threadIdx.x, nth = (mir ? nw - nwp : nwp) * 64;
    // ---- layout of the pool: the two GU, the two W, then one-node tables
    const int mult = STAGED ? M : 1, row_n = STAGED ? staged_row(M) : M + 1;
    const size_t gu = STAGED ? row_n : M;
    e.GU = e.pool;
    const unsigned atP = (unsigned)((bandP + bandS) * gu), sizeP = (unsigned)(band_size(bandP, lenP) * mult), used = atP + sizeP + (unsigned)(band_size(bandS, lenS) * mult);
    double *WP = e.pool + atP, *WS = WP + sizeP, *G = e.pool + used;
    const bool in_regs = REGS && e.ints[2] && imax(bandP, bandS) <= 64 && used <= e.pool_n; // node_tables()
    const unsigned table = in_regs ? 0u : (unsigned)(imax(bandP, bandS) + 1) * row_n;
    // ---- few nodes, each of many layers: tables over (layers covered, GPUs used) are smaller work than a table per start layer (nodes against
    // layers per node), and the covers next to the slowest stage are their last rows.  Against tables in LDS from four layers a node on.  Against
    // node_tables() from eight on, if bands are so wide that a wave holds one start or two: 64 layers x 8 GPUs, up to 2 nodes 581 -> 354 us (396 with LDS alone);
    // from bands of 16 on 40 layers x 4 GPUs, 2 nodes 94 -> 115 us; beyond 32 for eight GPUs too 48 layers, 2 nodes 344 -> 394 us; from twelve layers a
    // node on 52 layers x 8 GPUs, 3 nodes 393 -> 601 us.  Never with one or two GPUs per node, where node_tables() has hardly anything to add up, for a
    // single node, which has one start a side, or with stage counts, where rows over (GPUs, stages) are longer (34 layers x 8 GPUs, 3 nodes 247 -> 510 us).
    const int wide = imax(bandP, bandS);
    const bool by_gpus = !STAGED && M > 2 && nhi > 1 && nhi * 8 <= wide && wide > (M == 8 ? 24 : 32);
    if (!in_regs || by_gpus) {
        const int nd = imax(cendP, cendS) * M, jd = STAGED ? imin(J, nd + 1) : 1;
        const unsigned need = ((unsigned)lenP + 1 + lenS + 1) * nd * jd; // below 2^29
        if (nhi * 4 <= wide && need <= e.pool_n) {
            const int row_n = nd * jd;
            const int second = (lenP + 1) * row_n; // the other side's table
            for (int i = threadIdx.x; i < 2 * row_n; i += blockDim.x) {
                const int side = i >= row_n, o = i - side * row_n;
                e.pool[side * second + o] = o == 0 ? 0.0 : kNone;
            }
            wg_sync();
            for (int r = 1; r <= imax(lenP, lenS); ++r) {
                if (!mir) { if (r <= lenP) gpu_row<false, STAGED, MT, SUM, PAD>(a, e, r, nd, jd, tau, 1.0, ptau * tau, e.pool, th, nth); }
                else      { if (r <= lenS) gpu_row<true, STAGED, MT, SUM, PAD>(a, e, r, nd, jd, tau, 2.0, stau * tau, e.pool + second, th, nth); }
                wg_sync();
            }
            for (int i = threadIdx.x; i < (cendP + cendS) * M * J; i += blockDim.x) {
                const bool after = i >= cendP * M * J;
                const int o = after ? i - cendP * M * J : i, d0 = o / J, j = o - d0 * J;
                e.OUT[(after ? a.nodes * M * J : 0) + o] =
                    j < jd ? e.pool[(after ? second + lenS * row_n : lenP * row_n) + d0 * jd + j] : kNone;
            }
            wg_sync();
            combine<STAGED>(a, e, d, tau, nhi, cendP, cendS, mid, s_best);
            return true;
        }
    }
    if (used + table > e.pool_n) return false; // (without stage counts they fit: eval_pool())
    // ---- phase 1
    if constexpr (REGS) if (in_regs) {
        const int sP = 64 / imax(bandP, 1), sS = 64 / imax(bandS, 1); // start layers a wave takes at a time
        // (with a single node in all there is only the start at the far end)
        const int nP = nhi == 1 ? lenP > 0 : (lenP + sP - 1) / sP, nS = nhi == 1 ? lenS > 0 : (lenS + sS - 1) / sS, both = 2 * imin(nP, nS);
        for (int item = wave; item < nP + nS; item += nw) { // the two sides in turn
            int side, i;
            if (item < both) { side = item & 1; i = item >> 1; }
            else { side = nS > nP; i = item - (both >> 1); }
            if (!side) node_tables<false, STAGED, MT, PAD>(a, e, lenP, bandP, tau, 1.0, ptau * tau, WP, e.GU, i * sP, sP);
            else       node_tables<true, STAGED, MT, PAD>(a, e, lenS, bandS, tau, 2.0, stau * tau, WS, e.GU + bandP * gu, i * sS, sS);
        }
    }
    if (!in_regs) {
        const int fit = (int)((e.pool_n - used) / table); // one-node tables side by side
        int gbits = 0;
        while (1 << gbits < M) ++gbits;
        int lgxs = STAGED ? gbits : 0, slots = 64 >> (gbits + lgxs), waves = nw;
        if (slots > fit) {
            if (STAGED) slots = fit;
            else while (slots > 1 && slots > fit) { slots >>= 1; ++lgxs; }
        }
        // long walks of few tables: more lanes per walk rather than idle waves
        if (!STAGED) while (slots > 1 && slots * 4 > fit && imax(bandP, bandS) > 16) { slots >>= 1; ++lgxs; }
        // fewer tables for every wave, or as many for fewer waves: whichever are more (57 layers x 8 GPUs, 40 nodes 592 -> 514 us)
        const int each = imin(slots, fit / nw);
        if (!STAGED && each * nw > imin(nw, fit / slots) * slots) slots = each;
        waves = imin(waves, imax(1, fit / slots));
        if (wave < waves) {
            double *mine = G + (size_t)wave * slots * table;
            // (with a single node in all there is only the start at the far end)
            const int nP = nhi == 1 ? (lenP > 0) : (lenP + slots - 1) / slots, nS = nhi == 1 ? (lenS > 0) : (lenS + slots - 1) / slots, both = 2 * imin(nP, nS);
            for (int item = wave; item < nP + nS; item += waves) { // the two sides in turn
                int side, i;
                if (item < both) { side = item & 1; i = item >> 1; }
                else { side = nS > nP; i = item - (both >> 1); }
                if (!side) one_node_tables<false, STAGED, MT, SUM, PAD>(a, e, lenP, bandP, tau, 1.0, ptau * tau, WP, e.GU, mine, i * slots, slots, lgxs, gbits);
                else       one_node_tables<true, STAGED, MT, SUM, PAD>(a, e, lenS, bandS, tau, 2.0, stau * tau, WS, e.GU + bandP * gu, mine, i * slots, slots, lgxs, gbits);
            }
        }
    }
    // ---- phase 2: node after node, both sides at once.  Narrow bands: one wave each
    const unsigned histP = (unsigned)cendP * (bandP + 1), histS = (unsigned)cendS * (bandS + 1);
    if (!STAGED && imax(bandP, bandS) <= kChainBand && imax(lenP, lenS) <= kChainLen && used + histP + histS <= e.pool_n) {
        double *HP = G; // (in place of the one-node tables)
        wg_sync();
        if (wave == 0 || wave == nw - 1)
            node_chain_any(mir ? lenS : lenP, mir ? bandS : bandP, mir ? cendS : cendP, WP + (mir ? sizeP : 0), HP + (mir ? histP : 0));
        wg_sync();
        for (int i = threadIdx.x; i < (cendP + cendS) * M; i += blockDim.x) {
            const bool after = i >= cendP * M;
            const int o = after ? i - cendP * M : i, c = o / M, g = o - c * M, band = after ? bandS : bandP;
            const double *H = HP + (after ? histP : 0) + c * (band + 1), *cov = e.GU + (after ? bandP * M : 0) + g;
            double m = g == 0 ? H[0] : kNone;
            if (g > 0) for (int r = 1; r <= band; ++r) m = fmin(m, H[r] + cov[(r - 1) * M]);
            e.OUT[(after ? a.nodes * M : 0) + o] = m;
        }
        wg_sync();
    } else {
    // wide ones: half of the waves each (one side alone: all), a barrier per node count
    const bool alone = STAGED && (!lenP || !lenS), after = alone ? !lenP : (bool)mir;
    const int t0 = alone ? (int)threadIdx.x : th, tn = alone ? (int)blockDim.x : nth;
    double *cur = e.NP + (after ? (size_t)(lenP + 1) * J : 0), *nxt = cur + (size_t)(L + 2) * J;
    double *const out = e.OUT + (after ? (size_t)a.nodes * M * J : 0);
    const double *const W1 = WP + (after ? sizeP : 0), *const GU1 = e.GU + (after ? bandP * gu : 0);
    const int len = after ? lenS : lenP, band = after ? bandS : bandP, cend = after ? cendS : cendP;
    if constexpr (STAGED) {
        if (alone) node_out_staged<MT>(a, 0, 0, 0, cur, GU1, e.OUT + (after ? 0 : (size_t)a.nodes * M * J), t0, tn);
        wg_sync(); // W and GU are written
    } else {
        for (int i = th; i < len + 1; i += nth) { cur[i] = i == 0 ? 0.0 : kNone; nxt[i] = kNone; }
        wg_sync();
    }
    for (int c = 0; c < imax(cendP, cendS); ++c) {
        if (c < cend) {
            if constexpr (STAGED) {
                node_out_staged<MT>(a, len, band, c, cur, GU1, out, t0, tn);
                if (c + 1 < cend) node_step_staged<MT>(a, len, band, c, W1, cur, nxt, t0, tn);
            } else {
                node_out(M, len, band, c, cur, GU1, out, t0, tn);
                if (c + 1 < cend) node_step(len, band, c, W1, cur, nxt, t0, tn);
            }
        }
        wg_sync();
        double *t = cur; cur = nxt; nxt = t;
    }
    }
    combine<STAGED>(a, e, d, tau, nhi, cendP, cendS, mid, s_best);
    return true;
}

template <bool STAGED, int MT, bool SUM, bool PAD, bool REGS>
__global__ void __launch_bounds__(STAGED ? kStagedThreads : kEvalThreads, 4) k_exact_eval(Args a, int mode, int lds_doubles, int picks) {
    HIP_DYNAMIC_SHARED(double, s_dyn)
    __shared__ unsigned s_next;
    __shared__ int s_ints[4], s_nhi;
    const bool idle = *a.status != OOB_OK || !a.head->narrow; // the same for every thread: nothing is computed from a bad profile
    const int L = a.L, M = a.M, count = a.n_max - a.n_min + 1, J = STAGED ? a.Smax + 1 : 1, tid = threadIdx.x;
    if (idle) return;
    Eval e;
    e.pr = load_prof<SUM>(a, s_dyn, PAD ? a.M | 1 : a.M);
    // Places as whole numbers: a difference of pointers into LDS made every access of the pool a flat one (64 layers, 16 GPUs per node, one entry
    // 160 -> 194 us).
    unsigned at = (unsigned)prof_doubles(L, M, PAD ? M | 1 : M, SUM);
    e.reach = (unsigned char *)(s_dyn + at); at += (unsigned)(((size_t)(L + 1) * M + 7) / 8);
    e.NP = s_dyn + at;  at += 2 * (unsigned)(L + 2) * J;
    e.OUT = s_dyn + at; at += 2 * (unsigned)a.nodes * M * J;
    unsigned long long *s_best = (unsigned long long *)(s_dyn + at); at += a.live;
    e.pool = s_dyn + at; e.pool_n = (unsigned)lds_doubles - at;
    e.ints = s_ints;
    for (int i = tid; i < a.live; i += blockDim.x) s_best[i] = kNoneBits;
    const unsigned total = mode == kRest ? a.head->alive : a.head->ncand;
    if constexpr (REGS) {
        if (tid == 0) s_ints[2] = 1; // ends_ascend(), for node_tables()
        wg_sync();
        if (!ends_ascend<PAD>(e.pr, L, M)) s_ints[2] = 0;
    }
    for (int turn = 0;; ++turn) {
        wg_sync(); // the previous entry is done with LDS (and s_next has been read)
        unsigned c;
        int nhi = a.n_max;
        if (mode == kFirst) {
            // workgroup (template, rank): the bucket with the rank-th smallest bound for that template, its best entry
            if (turn) break;
            const int ni = (int)blockIdx.x / picks, pick = (int)blockIdx.x % picks;
            const int rank = pick * (pick + 1) / 2; // 0, 1, 3, 6, ...
            nhi = a.n_min + ni;
            const unsigned nb = a.head->nbuckets;
            float *key = (float *)e.pool;
            for (unsigned i = tid; i < nb; i += blockDim.x) key[i] = a.blb[(size_t)i * count + ni];
            if (tid == 0) s_next = 0xffffffffu;
            wg_sync();
            for (unsigned i = tid; i < nb; i += blockDim.x) {
                const float k = key[i];
                int below = 0;
                for (unsigned q = 0; q < nb; ++q) below += key[q] < k || (key[q] == k && q < i);
                if (below == rank && k < __builtin_huge_valf()) s_next = i * a.head->bucket + a.barg[(size_t)i * count + ni];
            }
            wg_sync();
            c = s_next;
            if (c == 0xffffffffu) break;
        } else {
            if (tid == 0) s_next = __hip_atomic_fetch_add(&a.head->next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid == 1) s_nhi = 0;
            wg_sync();
            c = s_next;
            if (c >= total) break; // every wave of every workgroup gets here
            if (mode == kAll) {
                // Without bounds of its own an entry is passed over if tau alone makes it too dear: of the j stages after it
                // each takes back at most tau, j <= the layers and GPUs after it (N_b given), or n stages cost at least
                // (3 n + 1) tau (N_b = 4 S).  The list ascends, so the first entries' minima meet the slow ones.
                const unsigned uvd = a.cuvd[c];
                const double tau = a.ctau[c];
                if (tid < a.live) { // (at most L <= 255: a thread each)
                    const int n = a.n_min + tid, j = imin(L - (int)(uvd >> 8 & 255), n * M - (int)(uvd >> 16));
                    const double least = a.Nb > 0 ? (double)imax(a.Nb - j, 0) * tau : (3.0 * n + 1.0) * tau;
                    if (least <= best_now(a, tid)) atomicMax(&s_nhi, n);
                }
                wg_sync();
                nhi = s_nhi;
                if (nhi == 0) continue;
            }
            if (mode == kRest) {
                c = a.list[c];
                // the minima may have fallen below this entry's bounds by now; n beyond the last template left is no use
                if constexpr (!STAGED) {
                    if (tid < a.live) {
                        const unsigned bk = c / a.head->bucket;
                        const double x = bound_of(a, a.lb + (size_t)c * a.nk, a.blo[bk], a.bfew[bk], a.n_min + tid);
                        if (x < kNone && x <= best_now(a, tid)) atomicMax(&s_nhi, a.n_min + tid);
                    }
                } else { // up to 64 multipliers: a lane per template and multiplier instead of a chain of reads per template
                    const unsigned bk = c / a.head->bucket;
                    const int lg = 32 - __clz(a.nk - 1), k = tid & ((1 << lg) - 1), per = (int)blockDim.x >> lg; // nk = 8 .. 64
                    const double lo = a.blo[bk];
                    const float lbk = k < a.nk ? a.lb[(size_t)c * a.nk + k] : 0.0f;
                    const int fewest = a.bfew[bk];
                    for (int n0 = 0; n0 < a.live; n0 += per) {
                        const int ni = n0 + (tid >> lg), n = a.n_min + ni;
                        double x = k < a.nk ? (double)lbk - lo * spent(a, k, n) : -kNone;
                        for (int d = 1; d < 1 << lg; d <<= 1) x = fmax(x, __shfl_xor(x, d, 64));
                        if (k == 0 && ni < a.live && n >= fewest && x < kNone && x <= best_now(a, ni)) atomicMax(&s_nhi, n);
                    }
                }
                wg_sync();
                nhi = s_nhi;
                if (nhi == 0) continue;
            }
        }
        if (!evaluate<STAGED, MT, SUM, PAD, REGS>(a, e, a.cuvd[c], a.ctau[c], nhi, s_best)) {
            // (not the first picks: the filter keeps those that matter, so each entry comes here once at most)
            if (STAGED && mode != kFirst && tid == 0) a.over[__hip_atomic_fetch_add(&a.head->over, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)] = c;
            continue;
        }
        if (mode != kFirst) { // let the other workgroups know
            wg_sync();
            for (int i = tid; i < a.live; i += blockDim.x)
                if (s_best[i] < (unsigned long long)__double_as_longlong(best_now(a, i))) atomicMin(&a.best[i], s_best[i]);
        }
    }
    wg_sync();
    for (int i = tid; i < a.live; i += blockDim.x)
        if (s_best[i] < (unsigned long long)__double_as_longlong(best_now(a, i))) atomicMin(&a.best[i], s_best[i]);
    if (mode != kFirst && !a.staged && last_workgroup(a)) finish(a, true); // (the staged entry point: k_exact_flat follows)
}

// ---------------------------------------------------------------------------------------------
// The general path: tables in the workspace.
//   Pre[p][D][j] = least sum over sequences covering [0, p) on exactly the first D GPUs (with j stages), t < tau
//   Suf[p][E][j] = the same for [p, L) on exactly the last E GPUs, t <= tau
// STAGED = false: J = 1, the sums carry the weights of the cost; STAGED = true: plain sums of t, the
// stage counts choose the coefficient of tau at the end and obey j1 + 1 + j2 <= N_b.
// After a fast path it takes the entries that path could not hold, and otherwise every stage.
// One workgroup takes one candidate slowest stage at a time (a grid-stride loop), walks the layers
// with two barriers per layer (the stage times into / out of the layer are staged in LDS), each
// thread owning (GPUs, stages) positions.
// Eight waves per SIMD are asked for: the up to kFlatSlots = 2 048 workgroups then run all at once.  Left to itself the compiler
// takes 106 scalar registers, which leaves seven, and the last eighth runs alone: 20.8 against 17.5 ms for 30 layers,
// 16 GPUs per node, 4 nodes, N_b = 20, and 64.0 against 48.3 ms for 60 layers, 2 nodes, N_b = 6.
// ---------------------------------------------------------------------------------------------
template <bool STAGED>
__global__ void __launch_bounds__(kThreads, 8) k_exact_flat(Args a) {
    HIP_DYNAMIC_SHARED(long long, s_flat) // [L * M] stage times into (or out of) the current layer, then [count] minima
    const int L = a.L, M = a.M, W = a.Dmax + 1, J = STAGED ? a.Smax + 1 : 1, count = a.n_max - a.n_min + 1;
    long long *s_col = s_flat, *s_best = s_flat + (size_t)L * M;
    const size_t plane = (size_t)W * J;
    long long *Pre = a.slots + (size_t)blockIdx.x * 2 * (L + 1) * plane, *Suf = Pre + (size_t)(L + 1) * plane;
    const long long *bnd = (const long long *)a.prof.boundary_ns;
    if (*a.status != OOB_OK) return;
    const bool narrow = a.head->narrow != 0; // a fast path has run: a.best holds doubles, and only its leftovers are to do
    if (narrow && a.head->over == 0) {
        if (blockIdx.x == 0) finish(a, true);
        return;
    }
    // time of stage [q, p) on dd GPUs, -1: impossible
    auto stage = [&](int q, int p, int dd) -> long long {
        if (q < a.flo[(size_t)p * M + dd - 1]) return -1;
        return a.PT[(size_t)p * M + dd - 1] - a.PT[(size_t)q * M + dd - 1] + (p < L ? bnd[p - 1] : 0);
    };
    const long long ptau = STAGED ? 0 : (a.Nb > 0 ? 0 : 4), stau = STAGED ? 0 : (a.Nb > 0 ? -1 : 3);
    const long long wsuf = STAGED ? 1 : 2;
    for (int i = threadIdx.x; i < count; i += kThreads) s_best[i] = kInf;
    const long long ncand = narrow ? (long long)a.head->over : (long long)L * (L + 1) / 2 * M;
    for (long long c = blockIdx.x; c < ncand; c += gridDim.x) {
        int u, v, d;
        if (narrow) { const unsigned x = a.cuvd[a.over[c]]; u = x & 255; v = x >> 8 & 255; d = x >> 16; }
        else triple((int)c, M, &u, &v, &d);
        const long long tau = stage(u, v, d);
        if (tau < 0) continue;
        wg_sync(); // the tables of the previous candidate are no longer read
        for (size_t i = threadIdx.x; i < plane; i += kThreads) Pre[i] = i == 0 ? 0 : kInf;
        for (int p = 1; p <= u; ++p) {
            wg_sync();
            for (int i = threadIdx.x; i < p * M; i += kThreads) // times of the stages [q, p) on dd GPUs
                s_col[i] = stage(i / M, p, i % M + 1);
            wg_sync();
            for (size_t i = threadIdx.x; i < plane; i += kThreads) {
                const int D = (int)(i / J), j = (int)(i % J);
                long long m = kInf;
                if (!STAGED || j >= 1)
                    for (int dd = 1; dd <= M && dd <= D; ++dd) {
                        const int D0 = D - dd;
                        if (D0 % M + dd > M) continue; // would cross a node boundary
                        const size_t src = (size_t)D0 * J + (STAGED ? j - 1 : 0);
                        for (int q = p - 1; q >= 0; --q) { // [q, p) only gets slower and heavier as q goes down
                            const long long tt = s_col[q * M + dd - 1];
                            if (tt < 0 || tt >= tau) break;
                            const long long x = Pre[(size_t)q * plane + src] + tt + ptau * tau;
                            m = x < m ? x : m;
                        }
                    }
                Pre[(size_t)p * plane + i] = m;
            }
        }
        wg_sync();
        for (size_t i = threadIdx.x; i < plane; i += kThreads) Suf[(size_t)L * plane + i] = i == 0 ? 0 : kInf;
        for (int p = L - 1; p >= v; --p) {
            wg_sync();
            for (int i = threadIdx.x; i < (L - p) * M; i += kThreads) // times of the stages [p, p+1+i/M) on dd GPUs
                s_col[i] = stage(p, p + 1 + i / M, i % M + 1);
            wg_sync();
            for (size_t i = threadIdx.x; i < plane; i += kThreads) {
                const int E = (int)(i / J), j = (int)(i % J);
                long long m = kInf;
                if (!STAGED || j >= 1)
                    for (int dd = 1; dd <= M && dd <= E; ++dd) {
                        const int E0 = E - dd;
                        if (E0 % M + dd > M) continue;
                        const size_t src = (size_t)E0 * J + (STAGED ? j - 1 : 0);
                        // [p, w) as w goes up: impossible stays impossible and the time without the boundary
                        // term only grows, so those end the loop; a stage that is only too slow because of
                        // the boundary term of its last layer is skipped, not the rest of the run
                        for (int w = p + 1; w <= L; ++w) {
                            const long long tt = s_col[(w - p - 1) * M + dd - 1];
                            if (tt < 0) break;
                            if (tt > tau) {
                                if (w == L || tt - bnd[w - 1] > tau) break;
                                continue;
                            }
                            const long long x = Suf[(size_t)w * plane + src] + wsuf * tt + stau * tau;
                            m = x < m ? x : m;
                        }
                    }
                Suf[(size_t)p * plane + i] = m;
            }
        }
        wg_sync();
        // the slowest stage at every place it fits, for every template
        for (size_t i = threadIdx.x; i < plane; i += kThreads) {
            const int D = (int)(i / J), j1 = (int)(i % J);
            if (D + d > a.Dmax) continue;
            if (D % M + d > M) continue;
            const long long pre = Pre[(size_t)u * plane + i];
            if (pre >= kInf / 2) continue;
            for (int n = a.n_min; n <= a.n_max; ++n) {
                const int E = n * M - D - d;
                if (E < 0) continue;
                if (!STAGED) {
                    if (!answered(a, n)) continue;
                    const long long suf = Suf[(size_t)v * plane + E];
                    if (suf >= kInf / 2) continue;
                    const long long tot = pre + (a.Nb > 0 ? (long long)a.Nb : 4ll) * tau + suf;
                    if (tot < s_best[n - a.n_min]) atomicMin((unsigned long long *)&s_best[n - a.n_min], (unsigned long long)tot);
                } else {
                    for (int j2 = 0; j1 + 1 + j2 <= a.Smax; ++j2) {
                        const long long suf = Suf[(size_t)v * plane + (size_t)E * J + j2];
                        if (suf >= kInf / 2) continue;
                        const long long coef = a.Nb > 0 ? (long long)a.Nb - j2 : 4ll * j1 + 4 + 3ll * j2;
                        const long long tot = pre + coef * tau + 2 * suf;
                        if (tot < s_best[n - a.n_min]) atomicMin((unsigned long long *)&s_best[n - a.n_min], (unsigned long long)tot);
                    }
                }
            }
        }
    }
    wg_sync();
    for (int i = threadIdx.x; i < count; i += kThreads)
        if (s_best[i] < kInf)
            atomicMin(&a.best[i], narrow ? (unsigned long long)__double_as_longlong((double)s_best[i]) : (unsigned long long)s_best[i]);
    if (last_workgroup(a)) finish(a, narrow);
}

inline size_t slot_bytes(int L, int Dmax, int J) { return align_up(sizeof(long long) * 2 * (size_t)(L + 1) * (Dmax + 1) * J); }

} // namespace oob_exact

static bool exact_dims_ok(int L, int n_max, int M) {
    return L >= 1 && L <= OOB_EXACT_MAX_L && n_max >= 1 && M >= 1 && M <= OOB_MAX_GPUS &&
           (long long)n_max * M <= OOB_EXACT_MAX_GPUS;
}
static int exact_smax(int L, int n_max, int M, int Nb) {
    int s = L < n_max * M ? L : n_max * M;
    return Nb > 0 && Nb < s ? Nb : s;
}

// The stage limit S <= N_b can bind for some template.
static bool exact_limit_binds(int L, int n_max, int M, int Nb) { return Nb > 0 && Nb < (L < n_max * M ? L : n_max * M); }

// LDS of the fast path, 0: none for this shape.
static oob_exact::EvalLds exact_lds(int L, int M, int n_max, int count, int Nb, bool staged) {
    if (!staged && !oob_exact::in_doubles(L, M, n_max, count)) return {0, false, false};
    const bool counts = staged && exact_limit_binds(L, n_max, M, Nb);
    return oob_exact::eval_lds(L, M, n_max, count, counts ? exact_smax(L, n_max, M, Nb) + 1 : 1, counts);
}

extern "C" size_t oob_exact_workspace_size(int L, int n_max, int gpus_per_node) {
    using namespace oob_exact;
    if (!exact_dims_ok(L, n_max, gpus_per_node)) return 0;
    const bool fast = exact_lds(L, gpus_per_node, n_max, n_max, 0, false).bytes != 0;
    size_t n = layout(L, gpus_per_node, n_max, fast, bound_mus(L, gpus_per_node, false), false).slots;
    if (!fast) n += (size_t)kFlatSlots * slot_bytes(L, n_max * gpus_per_node, 1); // tables beyond LDS: the general path
    return n;
}

extern "C" size_t oob_exact_staged_workspace_size(int L, int n_max, int gpus_per_node, int microbatches) {
    using namespace oob_exact;
    if (!exact_dims_ok(L, n_max, gpus_per_node) || microbatches < 0) return 0;
    const size_t slot = slot_bytes(L, n_max * gpus_per_node, exact_smax(L, n_max, gpus_per_node, microbatches) + 1);
    const size_t want = (size_t)1 << 30; // about a gigabyte of tables, at least 16 and at most kFlatSlots workgroups in flight
    size_t slots = want / slot;
    slots = slots < 16 ? 16 : slots > (size_t)kFlatSlots ? (size_t)kFlatSlots : slots;
    const int mus = bound_mus(L, gpus_per_node, exact_limit_binds(L, n_max, gpus_per_node, microbatches));
    return layout(L, gpus_per_node, n_max, exact_lds(L, gpus_per_node, n_max, n_max, microbatches, true).bytes != 0, mus, true).slots + slots * slot;
}

template <bool STAGED, int MT, bool SUM, bool PAD, bool REGS = MT != 0>
static int eval_launch_m(const oob_exact::Args &a, int mode, unsigned grid, int threads, size_t lds, int picks, hipStream_t st) {
    using namespace oob_exact;
    if (beyond_default(lds, kLdsStatic) && hipFuncSetAttribute((const void *)k_exact_eval<STAGED, MT, SUM, PAD, REGS>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return OOB_EHIP;
    hipLaunchKernelGGL((k_exact_eval<STAGED, MT, SUM, PAD, REGS>), dim3(grid), dim3(threads), lds, st, a, mode, (int)(lds / 8), picks);
    return OOB_OK;
}
template <bool STAGED> // a kernel of its own for the usual numbers of GPUs per node, known to the compiler
static int eval_launch(const oob_exact::Args &a, int mode, unsigned grid, int threads, size_t lds, int picks, hipStream_t st) {
    if constexpr (!STAGED) {
        if (a.sums) return eval_launch_m<false, 0, true, false>(a, mode, grid, threads, lds, picks, st);
        if (a.eval_pad) return eval_launch_m<false, 8, false, true>(a, mode, grid, threads, lds, picks, st); // can_pad()
    }
    if constexpr (STAGED) {
        if (!a.regs) return eval_launch_m<true, 8, false, false, false>(a, mode, grid, threads, lds, picks, st); // eval_tables_in_lds()
    }
    switch (a.M) {
    case 1: return eval_launch_m<STAGED, 1, false, false>(a, mode, grid, threads, lds, picks, st);
    case 2: return eval_launch_m<STAGED, 2, false, false>(a, mode, grid, threads, lds, picks, st);
    case 4: return eval_launch_m<STAGED, 4, false, false>(a, mode, grid, threads, lds, picks, st);
    case 8: return eval_launch_m<STAGED, 8, false, false>(a, mode, grid, threads, lds, picks, st);
    default: return eval_launch_m<STAGED, 0, false, false>(a, mode, grid, threads, lds, picks, st);
    }
}

template <int MT, bool PAD, bool MUS>
static int bounds_launch_m(const oob_exact::Args &a, int mus, size_t lds, hipStream_t st) {
    using namespace oob_exact;
    if (beyond_default(lds, kLdsStatic) && hipFuncSetAttribute((const void *)k_exact_bounds<MT, PAD, MUS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)lds) != hipSuccess)
        return OOB_EHIP;
    const unsigned nb = (unsigned)((tri(a.L) * a.M + bucket_least(a.nk) - 1) / bucket_least(a.nk));
    hipLaunchKernelGGL((k_exact_bounds<MT, PAD, MUS>), dim3(nb < (unsigned)kMaxBuckets ? nb : (unsigned)kMaxBuckets), dim3(kBoundThreads), lds, st, a, mus);
    return OOB_OK;
}
template <int MT, bool PAD>
static int bounds_launch(const oob_exact::Args &a, int mus, size_t lds, hipStream_t st) {
    return mus > 1 ? bounds_launch_m<MT, PAD, true>(a, mus, lds, st) : bounds_launch_m<MT, PAD, false>(a, mus, lds, st);
}

static int exact_launch(const oob_profile *profile, int L, int n_min, int n_max, int M, int microbatches, int64_t mem_cap,
                        void *dev_workspace, size_t workspace_bytes, int64_t *best, int32_t *status, void *stream,
                        bool staged) {
    using namespace oob_exact;
    if (!profile || !profile->fwd_ns || !profile->bwd_ns || !profile->mem_bytes || !profile->boundary_ns) return OOB_EINVAL;
    if (!best || !status || !dev_workspace || ((uintptr_t)dev_workspace & 255) != 0) return OOB_EINVAL;
    if (n_min < 1 || n_min > n_max || mem_cap <= 0 || microbatches < 0 || !exact_dims_ok(L, n_max, M)) return OOB_EINVAL;
    const int count = n_max - n_min + 1, Dmax = n_max * M;
    Args a;
    a.prof = *profile; a.L = L; a.M = M; a.n_min = n_min; a.n_max = n_max; a.Nb = microbatches; a.Dmax = Dmax;
    a.Smax = exact_smax(L, n_max, M, microbatches);
    a.cap = mem_cap;
    a.nodes = imin(n_max, L);
    a.top = staged || microbatches == 0 || microbatches >= L ? a.nodes : imin(a.nodes, microbatches / M); // as answered(): n M <= N_b
    a.live = imax(0, a.top - n_min + 1);
    // stage counts are only carried where the limit can bind
    const bool counts = staged && exact_limit_binds(L, n_max, M, microbatches);
    const int J = counts ? a.Smax + 1 : 1;
    const EvalLds ev = exact_lds(L, M, n_max, staged ? n_max : count, microbatches, staged); // (staged: as its workspace is sized)
    const size_t lds = ev.bytes;
    a.fast = lds != 0;
    a.sums = ev.sums;
    a.eval_pad = ev.pad && tri(L) * M > (size_t)kDirectMax; // (short models: 61 us either way, 62 padded, 15 layers)
    a.staged = staged;
    a.regs = !(counts && eval_tables_in_lds(L, M, n_max, J));
    const size_t ntri = tri(L) * M;
    const int mus = bound_mus(L, M, counts);
    a.bounds_pad = bound_pad(L, M, mus);
    a.bounds = a.fast && ntri > (size_t)kDirectMax && count <= kMaxCount && mus > 0;
    char *ws = (char *)dev_workspace;
    const Layout y = layout(L, M, n_max, a.fast, mus, staged);
    a.head = (Head *)(ws + y.head); a.PT = (long long *)(ws + y.PT); a.flo = (unsigned char *)(ws + y.flo);
    a.ctau = (double *)(ws + y.ctau); a.cuvd = (unsigned *)(ws + y.cuvd); a.lb = (float *)(ws + y.lb);
    a.blo = (double *)(ws + y.blo); a.bfew = (int *)(ws + y.bfew); a.nk = kLambdas * mus;
    a.blb = (float *)(ws + y.blb); a.barg = (unsigned short *)(ws + y.barg); a.list = (unsigned *)(ws + y.list);
    a.over = (unsigned *)(ws + y.over); a.slots = (long long *)(ws + y.slots);
    a.best = (unsigned long long *)best; a.status = status;
    hipStream_t st = (hipStream_t)stream;
    // the general path: shapes beyond LDS; with the staged entry point also times beyond 2^52 and entries beyond LDS
    const bool general = staged || !a.fast;
    size_t slots = 0;
    if (general) {
        const size_t slot = slot_bytes(L, Dmax, J);
        if (workspace_bytes < y.slots + 16 * slot) return OOB_ECAPACITY;
        slots = (workspace_bytes - y.slots) / slot;
        if (slots > (size_t)kFlatSlots) slots = kFlatSlots;
    } else if (workspace_bytes < y.slots) return OOB_ECAPACITY;
    a.limit = general ? kInf : kDoubleExact;
    const PrepLds prep = prep_lds(L, M, a.fast);
    if (beyond_default(prep.bytes, kPrepStatic) && hipFuncSetAttribute((const void *)k_exact_prep, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                                       (int)prep.bytes) != hipSuccess)
        return OOB_EHIP;
    hipLaunchKernelGGL(k_exact_prep, dim3(1), dim3(kPrepThreads), prep.bytes, st, a, prep.room);
    int rc = OOB_OK;
    if (a.fast) {
        const int threads = eval_threads(L, M, counts);
        const unsigned fill = (unsigned)(256 * imax(1, imin((int)(kLdsLimit / lds), 1024 / threads))); // workgroups the GPU holds at once
        if (a.bounds) {
            const size_t bl = 8 * bound_doubles(L, M, mus, a.bounds_pad);
            switch (M * 2 + a.bounds_pad) {
            case 2: rc = bounds_launch<1, false>(a, mus, bl, st); break;
            case 4: rc = bounds_launch<2, false>(a, mus, bl, st); break;
            case 8: rc = bounds_launch<4, false>(a, mus, bl, st); break;
            case 16: rc = bounds_launch<8, false>(a, mus, bl, st); break;
            case 17: rc = bounds_launch<8, true>(a, mus, bl, st); break;
            default: rc = bounds_launch<0, false>(a, mus, bl, st); break;
            }
            if (rc != OOB_OK) return rc;
            // no more than ten: the entries of the later ranks have the slow stages that take longest to evaluate (16: 584
            // instead of 372 us for 45 layers x 8 GPUs, 13 nodes, 754 instead of 481 us for 55 layers, 25 nodes)
            const int picks = imax(1, imin(10, (int)(fill / count)));
            rc = counts ? eval_launch<true>(a, kFirst, count * picks, threads, lds, picks, st)
                        : eval_launch<false>(a, kFirst, count * picks, threads, lds, picks, st);
            if (rc != OOB_OK) return rc;
            constexpr int per = kFilterThreads / 64 * kFilterEntries;
            hipLaunchKernelGGL(k_exact_filter, dim3((unsigned)((ntri + per - 1) / per)), dim3(kFilterThreads), 8 * (size_t)a.nk * a.live, st, a);
            rc = counts ? eval_launch<true>(a, kRest, fill, threads, lds, 0, st) : eval_launch<false>(a, kRest, fill, threads, lds, 0, st);
        } else {
            const unsigned some = fill < 512 ? fill : 512, grid = ntri < some ? (unsigned)ntri : some; // few enough to learn from each other
            rc = counts ? eval_launch<true>(a, kAll, grid, threads, lds, 0, st) : eval_launch<false>(a, kAll, grid, threads, lds, 0, st);
        }
        if (rc != OOB_OK) return rc;
    }
    if (general) {
        const unsigned grid = (unsigned)(ntri < slots ? ntri : slots);
        const size_t fl = sizeof(long long) * ((size_t)L * M + count);
        if (counts) hipLaunchKernelGGL(k_exact_flat<true>, dim3(grid), dim3(kThreads), fl, st, a);
        else        hipLaunchKernelGGL(k_exact_flat<false>, dim3(grid), dim3(kThreads), fl, st, a);
    }
    return hipGetLastError() == hipSuccess ? OOB_OK : OOB_EHIP;
}

extern "C" int oob_exact_minimum(const oob_profile *profile, int L, int n_min, int n_max, int gpus_per_node,
                                 int microbatches, int64_t mem_cap, void *dev_workspace, size_t workspace_bytes,
                                 int64_t *best, int32_t *status, void *stream) {
    return exact_launch(profile, L, n_min, n_max, gpus_per_node, microbatches, mem_cap, dev_workspace, workspace_bytes,
                        best, status, stream, false);
}

extern "C" int oob_exact_minimum_staged(const oob_profile *profile, int L, int n_min, int n_max, int gpus_per_node,
                                        int microbatches, int64_t mem_cap, void *dev_workspace, size_t workspace_bytes,
                                        int64_t *best, int32_t *status, void *stream) {
    return exact_launch(profile, L, n_min, n_max, gpus_per_node, microbatches, mem_cap, dev_workspace, workspace_bytes,
                        best, status, stream, true);
}
