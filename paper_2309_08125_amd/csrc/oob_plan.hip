// MI355X (gfx950) pipeline-template planner: kernels and host driver behind the C ABI of
// include/oob_plan.h.  Method: Section 4.1 of the Oobleck paper (node specification 4.1.1,
// GPU-stage mapping 4.1.2 with Eq. 1-4, coverage theorem of Appendix A).
//
// Arithmetic.  Inputs and outputs are int64.  Inside the tables every time is held as an
// IEEE double: gfx950 issues 64-bit floating add / min / compare at full rate (one VALU
// instruction each) while a 64-bit integer add or compare takes two or more, and doubles are
// exact for integers below 2^53.  The set-up kernel proves the bound (every quantity the
// recursion can form stays below 2^52 ns, about 52 days) or reports OOB_EOVERFLOW, so the
// results are bit-identical to int64 arithmetic in any evaluation order.
//
// What a state stores.  With r = S' - s and children A = (s, u, k, left set),
// B = (r, k, v, right set), Eq. 1-3 give the candidate's total
//     slowest stage in A (A.tmax >= B.tmax):  T = (A.T + cl * A.tmax) + 2 * B.T1
//     slowest stage in B:                     T = A.T1 + (B.T + cr * B.tmax)
// where X.T is the child's own total under its own stage count, and (cl, cr) = (-r, 0) when
// N_b is the caller's microbatch count or (3r, 4s) when N_b = 4 S' per state.  So the hot
// loop needs only (T, T1, tmax) per child: 2 adds (the second under a mask), 1 compare, 1 min per candidate.
// T3 and k* follow from the stages of a template and are formed for the templates alone (k_backtrack).
//
// One level S' = split kernels, then a select kernel.
//   k_split_key  per (block of the (u,v) plane, segment of its split points k, split s, group of
//            target device sets): the minimum over (k, m) of Eq. 1-3 per state as a
//            key of (total, s, k), merged into the level's key array (described at the kernel).
//            k_split is the variant without keys for shapes beyond its LDS.
//   k_level_small   both of these for a level of few candidates.
//   k_select_key / k_select  per state: from the smallest key (from the per-split minima) the first m at that
//            (s, k) whose candidate equals it -- the smallest (T, s, k, m) -- and the record.
// Before that one launch (k_prepare) scans and validates the profile, lays out the tables, lists the
// tasks of every level, clears the keys and does level 1; after the last level k_pick chooses the stage count of
// every template size, k_backtrack expands the stages and does Section 4.1.1's node specification.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
#include <algorithm>
#include <vector>
#include <math.h>
#include <new>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "oob_layout.h"
#include "oob_plan.h"

namespace oob {

constexpr double kNone = __builtin_huge_val(); // total of a state that does not exist
constexpr long long kExactBound = 1LL << 52;
constexpr int kInternalError = -5;             // status: a state's minimum was not re-found

struct Rec { double T, T1, tmax; long long choice; }; // 32 bytes, one per (table, u, v); the split that gives T: s | k << 10 | m << 21

// Device view of the workspace.
struct Tables {
    Shape sh;
    int NB;               // blocks per side of the (u, v) plane
    int coff;             // column shift of the plane: v sits in block column (v + coff) / 8
    int tab_recs;         // records per table = tri_blocks(NB) * 64
    int inv_M;            // over_M()
    Rec *rec;             // [tables * tab_recs]
    double *partT;        // [(S'-1) * deltas * tiles * 64] per-split minima of the current level
    unsigned long long *key; // the same memory: [deltas * tiles * 64] keys of the current level (keyed kernel)
    int *partK;           // same shape: first k reaching the minimum
    int2 *seg_tab;        // per level: (tile | split points << 16, ub | vb << 8 | offset of the first one << 16) of every split task
    int seg_stride;       // entries reserved per level in seg_tab (level S' starts at (S'-2) * seg_stride)
    int *flags;           // [0] 1: (total, k) keys fit a double and k_split_key runs
                          // [1] 1: the host chose the plain split kernel k_split for this job (then [0] = 0)
                          // [0] = [1] = 0: k_select evaluates every candidate itself
                          // [2], [3]: levels done by k_level_small, levels with splits on other streams (tests)
    int *status;
};

__device__ __forceinline__ Level level(const Tables &t, int S) { return level_of(S, t.sh.M, t.sh.n_max, t.inv_M); }
__device__ __forceinline__ long long rec_index(const Tables &t, int S, int delta, int u, int v) {
    return (long long)(level(t, S).base + delta) * t.tab_recs + rec_off(u, v, t.coff, t.NB);
}
// First record of block (ub, vb) of that table.
__device__ __forceinline__ long long rec_block(const Tables &t, int S, int delta, int ub, int vb) {
    return (long long)(level(t, S).base + delta) * t.tab_recs + (long long)tri_index(ub, vb, t.NB) * 64;
}

// ---------------------------------------------------------------------------------------
// Set-up: prefix sums (Eq. 4's sums become differences), input validation, level offsets.
// One workgroup of four waves: two of them scan the profile rows of d GPUs, 64 entries at a time (sums
// saturate, so that no input can overflow them; a saturated sum is reported, not used); one wave
// scans the bytes and the boundary terms, one lays out the levels.
// ---------------------------------------------------------------------------------------
constexpr int kSetupThreads = 256; // a larger workgroup waits long for a place on a GPU that other jobs of a batch keep busy

// Inclusive scan over the lanes of min(a + b, cap) for values in [0, cap], cap <= 2^62.
__device__ __forceinline__ unsigned long long scan_sat(unsigned long long x, unsigned long long cap, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(x, d, 64);
        if (lane >= d) { x += y; if (x > cap) x = cap; }
    }
    return x;
}
// Inclusive scan over the lanes of a whole wave by data-parallel moves (shifts within the rows of sixteen lanes, then the row sums
// handed on): a tenth of the time of shuffles through LDS.
__device__ __forceinline__ int scan_int(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
    return x;
}

// One wave scans the profile row of d GPUs: prefix sums of F + B and prefix counts of forbidden entries (Eq. 4's sums
// become differences).  Returns the row's sum; *bad collects what is wrong with the entries (1 negative, 2 too large).
__device__ __forceinline__ unsigned long long scan_times(const oob_profile &prof, int L, int M, int d, int lane, long long *PT, int *PF, int *bad) {
    const unsigned long long capT = (unsigned long long)kExactBound;
    unsigned long long carry = 0;
    int fcarry = 0;
    if (PT && lane == 0) { PT[0] = 0; PF[0] = 0; }
    for (int l0 = 0; l0 < L; l0 += 64) {
        const int l = l0 + lane;
        const bool in = l < L;
        const long long F = in ? prof.fwd_ns[(size_t)l * M + d - 1] : 0, B = in ? prof.bwd_ns[(size_t)l * M + d - 1] : 0;
        const bool neg = F < 0 || B < 0;
        const bool fb = F >= OOB_FORBIDDEN || B >= OOB_FORBIDDEN;
        const bool big = !neg && !fb && (F >= kExactBound || B >= kExactBound);
        if (neg) *bad = imax(*bad, 1);
        if (big) *bad = imax(*bad, 2);
        unsigned long long x = (neg || fb || big) ? 0ull : (unsigned long long)(F + B);
        if (x > capT) x = capT;
        x = scan_sat(x, capT, lane) + carry;
        if (x > capT) x = capT;
        const int c = scan_int(fb ? 1 : 0) + fcarry;
        if (PT && in) { PT[l + 1] = (long long)x; PF[l + 1] = c; }
        carry = __shfl(x, 63, 64);
        fcarry = __shfl(c, 63, 64);
    }
    return carry;
}
// The same for the bytes.
__device__ __forceinline__ unsigned long long scan_bytes(const oob_profile &prof, int L, int lane, long long *PM, int *bad) {
    const unsigned long long capM = (unsigned long long)OOB_FORBIDDEN;
    unsigned long long carry = 0;
    if (PM && lane == 0) PM[0] = 0;
    for (int l0 = 0; l0 < L; l0 += 64) {
        const int l = l0 + lane;
        const bool in = l < L;
        const long long mb = in ? prof.mem_bytes[l] : 0;
        const bool badm = mb < 0 || mb >= OOB_FORBIDDEN;
        if (badm) *bad = imax(*bad, 1);
        unsigned long long m = badm ? 0ull : (unsigned long long)mb;
        m = scan_sat(m, capM, lane) + carry;
        if (m > capM) m = capM;
        if (PM && in) PM[l + 1] = (long long)m;
        carry = __shfl(m, 63, 64);
    }
    return carry;
}

// How the host runs the levels, as one argument of the set-up launch (three of them cost it another wait for its
// arguments: 15.2 instead of 14.5 us): bit 0 the plain split kernel, then levels by k_level_small, levels on other streams.
constexpr int kHowBits = 15;
__device__ void setup_body(const Tables &t, const oob_profile &prof, int how) {
    const int L = t.sh.L, M = t.sh.M;
    __shared__ long long s_worst[OOB_MAX_GPUS + 1];
    __shared__ int s_bad;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    const unsigned long long capT = (unsigned long long)kExactBound, capM = (unsigned long long)OOB_FORBIDDEN;
    int bad = 0;
    for (int d = 1 + wave; d <= M && wave < nw - 2; d += nw - 2) { // row of d GPUs
        const unsigned long long sum = scan_times(prof, L, M, d, lane, nullptr, nullptr, &bad);
        if (sum >= capT) bad = imax(bad, 2);
        if (lane == 0) s_worst[d] = (long long)sum;
    }
    if (wave == nw - 2) { // bytes and boundary terms
        if (scan_bytes(prof, L, lane, nullptr, &bad) >= capM) bad = imax(bad, 1);
        unsigned long long cx = 0;
        for (int l0 = 0; l0 < L; l0 += 64) {
            const int l = l0 + lane;
            const long long xb = l < L ? prof.boundary_ns[l] : 0;
            if (xb < 0) bad = imax(bad, 1);
            if (xb >= kExactBound) bad = imax(bad, 2);
            unsigned long long x = (xb < 0 || xb >= kExactBound) ? 0ull : (unsigned long long)xb;
            x = scan_sat(x, capT, lane) + cx;
            if (x > capT) x = capT;
            cx = __shfl(x, 63, 64);
        }
        if (cx >= capT) bad = imax(bad, 2);
        if (lane == 0) s_worst[0] = (long long)cx;
    }
    if (bad) atomicMax(&s_bad, bad);
    __syncthreads();
    if (threadIdx.x == 0) {
        int st = OOB_OK, keys = 0;
        if (s_bad == 1) st = OOB_EINVAL;
        else if (s_bad == 2) st = OOB_EOVERFLOW;
        else {
            // Every quantity the recursion forms is at most (N_b + 4 Smax + 4) * w, where w bounds
            // the sum of all stage times of any pipeline; the sum over d of the row totals plus all
            // boundary terms is such a w (loose, never too small).
            long long worst = s_worst[0];
            for (int dd = 1; dd <= M; ++dd) {
                worst += s_worst[dd];
                if (worst >= kExactBound) worst = kExactBound;
            }
            const long long nb = t.sh.Nb > 0 ? t.sh.Nb : 4LL * t.sh.Smax;
            const long long mult = nb + 4LL * t.sh.Smax + 4;
            if (worst >= kExactBound / mult) st = OOB_EOVERFLOW;
            // a total and a split point k <= L fit one double as total * 2^kbits + k
            keys = st == OOB_OK && !(how & 1) && worst < (kExactBound >> key_bits(L)) / mult;
        }
        *(int4 *)t.flags = make_int4(keys, how & 1, how >> 1 & ((1 << kHowBits) - 1), how >> (1 + kHowBits));
        *t.status = st;
    }
}

// ---------------------------------------------------------------------------------------
// Level 1 ("Conquer", Eq. 4): stage time of layers [u, v) on d GPUs of one node (memory rule: ceil(bytes / d) <= cap;
// boundary term for a stage that is not the model's last).  Workgroup wg = (delta, four blocks of the plane), one wave
// per block, one lane per (u, v); it scans the two profile rows it needs for itself, which takes less time than waiting
// for another launch to have done it.
// ---------------------------------------------------------------------------------------
__device__ void level1_body(const Tables &t, const oob_profile &prof, int wg) {
    const int L = t.sh.L, M = t.sh.M, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ long long s_PT[OOB_MAX_L + 1], s_PM[OOB_MAX_L + 1];
    __shared__ int s_PF[OOB_MAX_L + 1];
    const int tiles = tile_count(L, 1), quads = (tiles + 3) / 4, delta = wg / quads, tile = (wg - delta * quads) * 4 + wave;
    const int d = delta < M - 1 ? delta + 1 : M;
    int bad = 0;
    if (wave == 0) scan_times(prof, L, M, d, lane, s_PT, s_PF, &bad);
    if (wave == 1) scan_bytes(prof, L, lane, s_PM, &bad);
    __syncthreads();
    if (tile >= tiles) return;
    int ub, vb;
    tile_decode(L, 1, tile, &ub, &vb);
    const int u = ub * 8 + (lane >> 3), v = vb * 8 + (lane & 7) - t.coff;
    Rec r = {kNone, kNone, 0.0, 0};
    if (u < L && v <= L && v - u >= 1 && s_PF[v] == s_PF[u]) { // (v < 0 in the first block column: no state)
        const long long bytes = s_PM[v] - s_PM[u];
        if ((bytes + d - 1) / d <= t.sh.cap) {
            const double nb = t.sh.Nb > 0 ? (double)t.sh.Nb : 4.0;
            r.T1 = r.tmax = (double)(s_PT[v] - s_PT[u] + (v < L ? prof.boundary_ns[v - 1] : 0));
            r.T = r.T1 + (nb - 2.0) * r.tmax + r.T1; // Eq. 2 with S' = 1, k* = 0, T3 = T1
        }
    }
    const long long o = (long long)delta * t.tab_recs + tri_index(ub, vb, t.NB) * 64 + lane; // level 1 has the first tables
    t.rec[o] = r;
}

// ---------------------------------------------------------------------------------------
// Levels S' >= 2 ("Divide", Eq. 1-3), first kernel: per (s, state) the minimum over (k, m).
//   grid.x  block (ub, vb) of the plane      grid.y  s - 1      grid.z  group of 8*waves sets
//   fam     0: targets inside one node (units = GPUs), 1: whole-node targets (units = nodes)
// PC = k values staged per pass.
// ---------------------------------------------------------------------------------------
template <int PC>
__global__ void __launch_bounds__(512) k_split(Tables t, int Sp, int fam, int NT, int NAall) {
    HIP_DYNAMIC_SHARED(double2, s_pair) // [ntab][PC][8] (x, y) pairs, then double tmax[ntab][PC][8]
    if (t.flags[1] == 0) return;        // only when the host chose this kernel (it then launches no other)
    const int L = t.sh.L, M = t.sh.M, n_max = t.sh.n_max;
    const int s = blockIdx.y + 1, r = Sp - s;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int ul = lane >> 3, vl = lane & 7;
    int ub, vb;
    tile_decode(L, Sp, blockIdx.x, &ub, &vb);
    const int fam_base = fam ? M - 2 : -1;
    int t_lo, t_hi;
    target_units(fam, Sp, M, n_max, &t_lo, &t_hi);
    const int a_wg0 = t_lo + blockIdx.z * nw * 8, a_wg1 = imin(t_hi, a_wg0 + nw * 8 - 1);
    int A_lo, A_hi, B_lo, B_hi;
    child_units(fam, s, M, n_max, &A_lo, &A_hi);
    child_units(fam, r, M, n_max, &B_lo, &B_hi);
    // left / right unit counts some target of this workgroup pairs up
    const int mA0 = imax(A_lo, a_wg0 - B_hi), mA1 = imin(A_hi, a_wg1 - B_lo);
    const int mB0 = imax(B_lo, a_wg0 - A_hi), mB1 = imin(B_hi, a_wg1 - A_lo);
    const int kmin = ub * 8 + s, kmax = tile_vmax(L, vb) - r;
    const bool work = mA0 <= mA1 && mB0 <= mB1 && kmin <= kmax;
    const int nA = work ? mA1 - mA0 + 1 : 0, nB = work ? mB1 - mB0 + 1 : 0, dummy = nA + nB;
    constexpr int TS = PC * 8;
    double *s_tm = (double *)(s_pair + (size_t)(dummy + 1) * TS);

    // this wave's targets a0..a0+7 and the left unit counts they use
    const int a0 = a_wg0 + wave * 8, a1 = imin(a_wg1, a0 + 7);
    const int mw0 = imax(mA0, a0 - B_hi), mw1 = imin(mA1, a1 - B_lo);
    const bool wave_work = work && a0 <= a_wg1 && mw0 <= mw1;

    double best[8];
    int bestk[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) { best[q] = kNone; bestk[q] = 0; }

    if (work) {
        for (int e = threadIdx.x; e < TS; e += blockDim.x) { // the "no such table" slot
            s_pair[dummy * TS + e] = make_double2(kNone, kNone);
            s_tm[dummy * TS + e] = 0.0;
        }
        const double cl = t.sh.Nb > 0 ? -(double)r : 3.0 * r, cr = t.sh.Nb > 0 ? 0.0 : 4.0 * s;
        const long long tabA = level(t, s).base + fam_base, tabB = level(t, r).base + fam_base;
        const int fillA = nA * TS, fill = (nA + nB) * TS;
        for (int kc = (kmin / PC) * PC; kc <= kmax; kc += PC) {
            __syncthreads(); // previous pass fully consumed
            for (int e = threadIdx.x; e < fill; e += blockDim.x) {
                if (e < fillA) {       // left child (s, u, k, m): row u of block (ub, k/8)
                    const int tab = e / TS, rem = e - tab * TS, u_l = rem / PC, k_l = rem - u_l * PC;
                    const int k = kc + k_l;
                    const Rec a = t.rec[(tabA + mA0 + tab) * t.tab_recs + (long long)tri_index(ub, (k + t.coff) >> 3, t.NB) * 64 +
                                        (u_l << 3) + ((k + t.coff) & 7)];
                    const int o = (tab * PC + k_l) * 8 + u_l;
                    s_pair[o] = make_double2(a.T + cl * a.tmax, a.T1);
                    s_tm[o] = a.tmax;
                } else {               // right child (r, k, v, m'): row k of block (k/8, vb)
                    const int e2 = e - fillA, tab = e2 / TS, rem = e2 - tab * TS, k_l = rem >> 3, v_l = rem & 7;
                    const int k = kc + k_l;
                    const Rec b = t.rec[(tabB + mB0 + tab) * t.tab_recs + (long long)tri_index(k >> 3, vb, t.NB) * 64 +
                                        ((k & 7) << 3) + v_l];
                    const int o = ((nA + tab) * PC + k_l) * 8 + v_l;
                    s_pair[o] = make_double2(2.0 * b.T1, b.T + cr * b.tmax);
                    s_tm[o] = b.tmax;
                }
            }
            __syncthreads();
            if (!wave_work) continue;
#pragma unroll 1
            for (int kl = 0; kl < PC; ++kl) {
                const int k = kc + kl;
                if (k < kmin || k > kmax) continue;
                double cur[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) cur[q] = kNone;
#pragma unroll 1
                for (int mm = mw0; mm <= mw1; mm += 8) {
                    double apa[8], at1[8], atm[8], bb2[15], bbt[15], btm[15];
#pragma unroll
                    for (int qm = 0; qm < 8; ++qm) {
                        const int m = mm + qm;
                        const int tab = m <= mA1 ? m - mA0 : dummy;
                        const int o = (tab * PC + kl) * 8 + ul;
                        const double2 p = s_pair[o];
                        apa[qm] = p.x; at1[qm] = p.y; atm[qm] = s_tm[o];
                    }
#pragma unroll
                    for (int d = 0; d < 15; ++d) {
                        const int mp = a0 - mm - 7 + d; // m' = (a0 + qa) - (mm + qm), d = qa - qm + 7
                        const int tab = (mp >= mB0 && mp <= mB1) ? nA + mp - mB0 : dummy;
                        const int o = (tab * PC + kl) * 8 + vl;
                        const double2 p = s_pair[o];
                        bb2[d] = p.x; bbt[d] = p.y; btm[d] = s_tm[o];
                    }
#pragma unroll
                    for (int qm = 0; qm < 8; ++qm)
#pragma unroll
                        for (int qa = 0; qa < 8; ++qa) {
                            const int d = qa - qm + 7;
                            const double T = atm[qm] >= btm[d] ? apa[qm] + bb2[d] : at1[qm] + bbt[d];
                            cur[qa] = fmin(cur[qa], T);
                        }
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) { // first k that reaches the minimum
                    const bool lt = cur[q] < best[q];
                    best[q] = lt ? cur[q] : best[q];
                    bestk[q] = lt ? k : bestk[q];
                }
            }
        }
    }
    if (a0 <= a_wg1) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (a0 + q > a_wg1) break;
            const int aidx = fam_base + a0 + q - dlo_of(Sp, M);
            const long long slot = ((long long)(s - 1) * NAall + aidx) * NT + blockIdx.x;
            t.partT[slot * 64 + lane] = best[q];
            t.partK[slot * 64 + lane] = bestk[q];
        }
    }
}

// ---------------------------------------------------------------------------------------
// Levels S' >= 2, first kernel, keyed variant (runs when flags[0] = 1).
//
// Same result as k_split, different mapping.  A workgroup owns (block of the plane, segment of
// its split points, s) and a group of up to kKeyTargets target sets; each of its waves takes every nw-th split point k
// of the segment for itself: it stages the streaming child's records for every unit count it needs in LDS, and the
// other child's eight unit counts at a time.  The (m, m') pairs of a split form a rectangle; an item keeps eight records
// of one side in registers (the STATIONARY side, cut into blocks of eight unit counts, the last one padded) and
// streams the other side.  Which child is stationary is chosen per workgroup so that the padding is smaller (it is the
// same work either way).  A step forms eight candidates, which belong to eight consecutive targets.  The eight running
// minima rotate: after a step the minimum of the lowest target is complete for this item and is merged into the
// workgroup's LDS table acc[a][lane] with an integer atomic min on the bits of key = total * 2^kbits + k
// (non-negative doubles order like their bit patterns).  The key makes the merge order-free
// and yields, per (s, state), the smallest total and the first k reaching it at once.  At the end the workgroup merges
// its keys, with the split in them, into the level's key per state: one key to read for the select where there
// was one per split, and two orders of magnitude less memory to clear (batch of 32 jobs 99 -> 95 ms, headline
// workload 8.43 -> 8.28 ms; reading the key first to save the atomic costs more than the atomic: 103 ms; eight or
// sixteen keys per state against contention 96.6 and 97.8 ms).
//
// What bounds it: the instructions a wave issues, and its waits.  The step loop alone, out of LDS, takes 175 cycles of
// a SIMD a step (eight candidates of 64 lanes) with four waves per SIMD, 186 with three, 206 with two, and about ten
// steps make an item.  When the four waves of a workgroup shared a split point they staged it together between two
// barriers and did about five steps each between them: as many scalar as vector instructions, half of the vector
// ones outside the steps, 40 % of a wave's time in waits.  A split point per wave has no barrier between set-up and
// merge, no item cut in pieces and a quarter of the scalar work, and pays with LDS for a streaming side per wave; the
// stationary side needs LDS for one block only and is loaded while the block before is worked on.  Measured: batch of 32
// jobs of 24..128 layers 124 -> 99 ms; staged by the workgroup four split points at a time with eight waves 149 ms; both
// children staged per wave 113 ms; three waves per workgroup 101 ms.
// Then what decides is how many waves share a compute unit.  The key table has a row per target and none beside them
// (minima of targets outside the group are dropped instead of collected in seven padding rows on either side), the
// staged side is as long as it is, and the kernel holds 128 registers without spills for four waves per SIMD: lane offsets
// of the staging are formed where they are used, and one eight of streaming tables is in flight instead of three.
// Batch 96 -> 79 ms, headline workload 7.36 -> 6.86 ms, 61 layers 1.30 -> 1.19 ms.  (Padding rows in classes of six
// rows and three waves per SIMD: 87 and 7.06 ms; five spilled registers: 83 and 7.17 ms, and 4 us a launch; the
// groups of four candidates whose select is the same in all lanes done by an add and a min, 57-77 % of them: 103 and
// 8.4 ms, the branches to them cost more than they save.)
// ---------------------------------------------------------------------------------------
constexpr int kKeyTargets = 64;
constexpr int kFillBatch = 1; // eights of streaming tables a wave has in flight while it works on the split point before
constexpr int kWavesPerSimd = 4;

// Workgroup x of a launch of n -> position in the task list (handle option OOB_OPT_XCD_ORDER only).  The hardware
// deals consecutive workgroups out to the 8 XCDs in turn; this hands every XCD one contiguous
// stretch of the list instead (workgroups x, x + 8, x + 16, ... walk it in order), so that tasks
// that share records meet in one L2.  A bijection on 0..n-1 for any n.  Measured on the headline
// workload: 29 % fewer bytes fetched from HBM, but 2 % more time (the stretches are not equally
// heavy and the kernel is bound by the vector ALUs), hence off by default.
__device__ __forceinline__ int xcd_chunked(int x, int n) {
    const int c = x & 7, i = x >> 3, q = n >> 3, rem = n & 7;
    return c * q + imin(c, rem) + i;
}

struct Rec24 { double2 a; double tm; }; // (T, T1), tmax: the 24 bytes of a record the splits need

// Which child streams: the one that leaves less padding when the other one is cut into blocks of eight, but none of
// more than `cap` tables.
__host__ __device__ __forceinline__ bool left_streams(int nA, int nB, int cap) {
    const bool left = nA * ((nB + 7) & ~7) <= nB * ((nA + 7) & ~7);
    return left == ((left ? nA : nB) <= cap);
}
__device__ __forceinline__ int log2_up(int x) { return 32 - __clz(x - 1); } // smallest b with 2^b >= x, x >= 1

// Four candidates of a step: streaming record (p, atm) against four stationary ones, into the minima a0..a3
// (LAST: a3 starts with its candidate).  The kernel is bound by the instructions its waves issue.  Written as a
// compare and a select a candidate takes 6 vector instructions (a 64-bit select is two, and two idle slots before
// them wait for the mask); here the sum of the other side overwrites the first one under the mask of the lanes that
// take it: 4 vector instructions and a move on the scalar unit.  Measured: headline workload 9.03 -> 8.35 ms a call,
// batch of 32 jobs 134 -> 124 ms, 61 layers 2.38 -> 2.29 ms.
template <bool LAST>
__device__ __forceinline__ void four_candidates(double &a0, double &a1, double &a2, double &a3, const double *bb2, const double *bbt,
                                                const double *btm, const double2 p, const double atm) {
    double t0, t1, t2;
    unsigned long long m0, m1, m2, m3, ex;
#define OOB_MIN3 "v_min_f64 %[a0], %[a0], %[t0]\n v_min_f64 %[a1], %[a1], %[t1]\n v_min_f64 %[a2], %[a2], %[t2]\n"
#define OOB_FOUR(T3, MIN3)                                                                                             \
    asm("v_cmp_lt_f64 %[m0], %[tm], %[c0]\n v_cmp_lt_f64 %[m1], %[tm], %[c1]\n"                                          \
        "v_cmp_lt_f64 %[m2], %[tm], %[c2]\n v_cmp_lt_f64 %[m3], %[tm], %[c3]\n s_mov_b64 %[ex], exec\n"                  \
        "v_add_f64 %[t0], %[px], %[x0]\n v_add_f64 %[t1], %[px], %[x1]\n v_add_f64 %[t2], %[px], %[x2]\n v_add_f64 " T3 ", %[px], %[x3]\n" \
        "s_mov_b64 exec, %[m0]\n v_add_f64 %[t0], %[py], %[y0]\n s_mov_b64 exec, %[m1]\n v_add_f64 %[t1], %[py], %[y1]\n" \
        "s_mov_b64 exec, %[m2]\n v_add_f64 %[t2], %[py], %[y2]\n s_mov_b64 exec, %[m3]\n v_add_f64 " T3 ", %[py], %[y3]\n" \
        "s_mov_b64 exec, %[ex]\n" OOB_MIN3 MIN3
#define OOB_FOUR_IN                                                                                                    \
    [px] "v"(p.x), [py] "v"(p.y), [tm] "v"(atm), [x0] "v"(bb2[0]), [x1] "v"(bb2[1]), [x2] "v"(bb2[2]), [x3] "v"(bb2[3]), \
        [y0] "v"(bbt[0]), [y1] "v"(bbt[1]), [y2] "v"(bbt[2]), [y3] "v"(bbt[3]), [c0] "v"(btm[0]), [c1] "v"(btm[1]),      \
        [c2] "v"(btm[2]), [c3] "v"(btm[3])
    if (LAST) {
        OOB_FOUR("%[a3]", "")
            : [a0] "+v"(a0), [a1] "+v"(a1), [a2] "+v"(a2), [a3] "=&v"(a3), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [m0] "=&s"(m0),
              [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3), [ex] "=&s"(ex)
            : OOB_FOUR_IN : "scc");
    } else {
        double t3;
        OOB_FOUR("%[t3]", "v_min_f64 %[a3], %[a3], %[t3]\n")
            : [a0] "+v"(a0), [a1] "+v"(a1), [a2] "+v"(a2), [a3] "+v"(a3), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [m0] "=&s"(m0),
              [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3), [ex] "=&s"(ex)
            : OOB_FOUR_IN : "scc");
    }
#undef OOB_FOUR
#undef OOB_FOUR_IN
#undef OOB_MIN3
}

// A keyed launch (level, families, splits); filled in by the host.
struct KeyArgs {
    int Sp, fam0, gz;    // the first gz target groups of the launch belong to family fam0, the rest (a launch that covers
                         // both families of a low level) to the whole-node family
    int NT;
    int s0, sstep;       // a launch covers the splits s0, s0 + sstep, ...
    int na;              // rows of the key table: targets of the largest group
    int cap;             // most streaming tables of a split point
    int t_lo1, dlo;      // smallest target of the whole-node family; first device set of the level
    int pack, xcd;       // several items per wave near the range ends; XCD-chunked task order
};

// Key of a level: total, split and split point as one integer, so that the smallest key is the smallest (T, s, k).  The
// key of a workgroup is total * 2^kb + k below 2^52 in a double; s and k take kb <= 10 bits each.
constexpr unsigned long long kNoKey = 0x7FF0000000000000ull;

__device__ __forceinline__ unsigned long long wide_key(double part, int s, int kb) {
    const unsigned long long v = (unsigned long long)__double_as_longlong(part + 0x1p52) & ((1ull << 52) - 1);
    return (((v >> kb) << kb | (unsigned)s) << kb) | (v & ((1ull << kb) - 1));
}

// A value that is the same in all lanes, in scalar registers.
__device__ __forceinline__ double uniform(double x) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)), __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// Order of a wave's LDS operations against those of its other lanes (they execute in order: only the compiler has to
// be told).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ Rec24 load24(const void *base, unsigned off) {
    const Rec *p = (const Rec *)((const char *)base + off);
    Rec24 rc;
    rc.a = *(const double2 *)p;
    rc.tm = p->tmax;
    return rc;
}

__global__ void __launch_bounds__(256, kWavesPerSimd) k_split_key(Tables t, KeyArgs ka) {
    // the launch's LDS: [na of the launch * 64] keys, row = target; then per wave [TS] pre-combined pairs, [TS] tmax
    // (negated when the right child streams)
    HIP_DYNAMIC_SHARED(unsigned long long, s_acc)
    const int Sp = ka.Sp, s = ka.s0 + blockIdx.y * ka.sstep, r = Sp - s;
    const int2 sg = t.seg_tab[(long long)(Sp - 2) * t.seg_stride + (ka.xcd ? xcd_chunked(blockIdx.x, gridDim.x) : (int)blockIdx.x)];
    const Level dA = level(t, s), dB = level(t, r);
    if (t.flags[0] == 0) return;        // keys do not fit: k_select evaluates the candidates itself
    const int L = t.sh.L, M = t.sh.M, n_max = t.sh.n_max;
    // the wave index is the same in all lanes: say so, and everything derived from it (work item,
    // m range, key row) is scalar arithmetic and scalar branches
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int tile = sg.x & 0xffff, klen = sg.x >> 16, ub = sg.y & 255, vb = (sg.y >> 8) & 255, kofs = sg.y >> 16;
    const int fam = (int)blockIdx.z < ka.gz ? ka.fam0 : 1, zg = (int)blockIdx.z < ka.gz ? (int)blockIdx.z : (int)blockIdx.z - ka.gz;
    const int fam_base = fam ? M - 2 : -1;
    const int a_g0 = (fam ? ka.t_lo1 : Sp) + zg * kKeyTargets, a_g1 = imin(fam ? imin(Sp, n_max) : M, a_g0 + kKeyTargets - 1);
    const int na = a_g1 - a_g0 + 1;
    const int A_lo = fam ? dA.least : s, A_hi = fam ? imin(s, n_max) : M - 1, B_lo = fam ? dB.least : r, B_hi = fam ? imin(r, n_max) : M - 1;
    const int mA0 = imax(A_lo, a_g0 - B_hi), mA1 = imin(A_hi, a_g1 - B_lo);
    const int mB0 = imax(B_lo, a_g0 - A_hi), mB1 = imin(B_hi, a_g1 - A_lo);
    const int vmax = tile_vmax(L, vb); // last layer position of the block's columns (never beyond L)
    const int kmin = ub * 8 + s + kofs, kmax = imin(vmax - r, kmin + klen - 1); // this workgroup's segment of the block's split points
    if (!(mA0 <= mA1 && mB0 <= mB1 && kmin <= kmax)) return; // nothing to merge
    const bool y_left = left_streams(mA1 - mA0 + 1, mB1 - mB0 + 1, ka.cap);
    const int yM0 = y_left ? mA0 : mB0, yM1 = y_left ? mA1 : mB1; // streaming unit counts
    const int qM0 = y_left ? mB0 : mA0, qM1 = y_left ? mB1 : mA1; // stationary unit counts
    const int nY = yM1 - yM0 + 1, nS = qM1 - qM0 + 1, nyb = (nY + 7) >> 3, nmb = (nS + 7) >> 3;
    const int fillY = nY * 8, TS = fillY + 64; // records staged: the streaming side of a split point, one block of the stationary side
    const unsigned long long kNoneBits = 0x7FF0000000000000ull;
    const double KS = uniform((double)(1 << key_bits(L)));

    // Staging.  The left child (s, u, k, m) is row u of block (ub, k/8), column k; the right child (r, k, v, m') is row
    // k of block (k/8, vb), column v.  What depends on the lane does not depend on k: eight tables ahead is a constant
    // distance, and only the last eight tables of a side may not all exist (streaming: the last one again, stationary:
    // "no such state").
    const double cl = uniform(t.sh.Nb > 0 ? -(double)r : 3.0 * r), cr = uniform(t.sh.Nb > 0 ? 0.0 : 4.0 * s);
    const long long tabA = (long long)(dA.base + fam_base + mA0) * t.tab_recs, tabB = (long long)(dB.base + fam_base + mB0) * t.tab_recs;
    const Rec *const recY = t.rec + (y_left ? tabA : tabB), *const recS = t.rec + (y_left ? tabB : tabA);
    const int lt = lane >> 3, li = lane & 7, shY = y_left ? 3 : 0, shS = y_left ? 0 : 3;
    auto off8 = [=](int sh, int top) { // lane's record of eight tables 0..top
        int ln = lane;
        asm volatile("" : "+v"(ln)); // formed where it is used: kept across the split points these offsets cost registers the kernel does not have
        return (__umul24(imin(ln >> 3, top), t.tab_recs) + ((ln & 7) << sh)) * 32u;
    };
    const int lastY = nY - 1 - 8 * (nyb - 1); // last table of the last eight of the streaming side that exists
    const int last = nS - 1 - 8 * (nmb - 1); // last table of the last stationary block that exists
    const size_t step8 = (size_t)t.tab_recs * 8 * sizeof(Rec);
    double2 *const pair = (double2 *)(s_acc + ka.na * 64) + wave * (TS + TS / 2);
    double *const tmv = (double *)(pair + TS);
    struct Src { const char *y, *s; };
    auto source = [=](int k) { // records of split point k of the two sides' first tables
        const int ck = k + t.coff; // column of split point k in the left child's table
        const int offL = tri_index(ub, ck >> 3, t.NB) * 64 + (ck & 7), offR = tri_index(k >> 3, vb, t.NB) * 64 + ((k & 7) << 3);
        return Src{(const char *)(recY + (y_left ? offL : offR)), (const char *)(recS + (y_left ? offR : offL))};
    };
    // Staged values are pre-combined with the level's coefficients: left records as (T + cl tmax, T1), right records as
    // (2 T1, T + cr tmax).  The slowest-stage test of Eq. 3 is "left tmax >= right tmax"; the step loop always tests
    // "streaming >= stationary", so when the right child streams both tmax are stored negated.
    auto combine = [=](const Rec24 &rc, bool left) {
        return Rec24{left ? make_double2(rc.a.x + cl * rc.tm, rc.a.y) : make_double2(2.0 * rc.a.y, rc.a.x + cr * rc.tm), y_left ? rc.tm : -rc.tm};
    };
    auto store = [=](int at, const Rec24 &rc) { pair[at] = rc.a; tmv[at] = rc.tm; };
    auto storeY = [=](int i, const Rec24 &rc) { // eight tables of the streaming side, those that exist
        if (i < nyb - 1 || lt <= lastY) store(i * 64 + lane, combine(rc, y_left));
    };

    Rec24 preY[kFillBatch], preS; // in flight: streaming side of the next split point, next stationary block
    int k = kmin + wave;
    auto loadY = [=](const Src &src, int i) { return load24(src.y + i * step8, off8(shY, i == nyb - 1 ? lastY : 7)); };
    auto loadS = [=](const Src &src, int i) { return load24(src.s + i * step8, off8(shS, i == nmb - 1 ? last : 7)); };
    if (k <= kmax) {
        const Src src = source(k);
#pragma unroll
        for (int i = 0; i < kFillBatch; ++i)
            if (i < nyb) preY[i] = loadY(src, i);
        preS = loadS(src, 0);
    }
    for (int e = threadIdx.x; e < na * 64; e += blockDim.x) s_acc[e] = kNoneBits;
    __syncthreads();
    for (; k <= kmax; k += nw) {
        const Src src = source(k);
#pragma unroll
        for (int i = 0; i < kFillBatch; ++i)
            if (i < nyb) storeY(i, preY[i]);
        for (int i = kFillBatch; i < nyb; ++i) storeY(i, loadY(src, i));
        const Src next = source(imin(k + nw, kmax));
        if (k + nw <= kmax) { // records of this wave's next split point: in flight during this one
#pragma unroll
            for (int i = 0; i < kFillBatch; ++i)
                if (i < nyb) preY[i] = loadY(next, i);
        }
        wave_fence();
        // Work items: the 8-blocks of the stationary side, 2^lgR of them side by side.
        // Only the rows 0..jr of the block hold states that can be split at k (u + s <= k), and only the
        // columns 7-jc..7 (k <= v - r; a block column that is not full lacks its first columns): near the ends
        // of the block's split range most of the 64 states idle.  Then the wave takes R items at once: the rows (or
        // columns) that matter, padded to a power of two, times R stationary blocks.
        const int jr = k - (ub * 8 + s), jc = vmax - r - k;
        const int lr = log2_up(imin(jr, 7) + 1), lc = log2_up(imin(jc, 7) + 1);
        const int lgR = ka.pack && nmb > 1 ? 3 - imin(lr, lc) : 0;
        const int nsup = (nmb + (1 << lgR) - 1) >> lgR;
        const double kd = (double)k;
        // One item, with (PACK) or without several stationary blocks side by side in the wave; the plain variant
        // keeps the item's block and row offset in scalar registers.
        auto run = [&](auto pack_c, const int sb, const int slot, const int ue, const int ve) {
            constexpr bool PACK = decltype(pack_c)::value;
            const int yl = y_left ? ue : ve, ql = y_left ? ve : ue; // lane index of a streaming / stationary record
            const int col = PACK ? ue * 8 + ve : lane;              // this lane's state: its column of the key table
            // stationary blocks mb_first .. mb_last (those that exist); this lane's is mb.  A lane without a
            // block of its own repeats the last block's work for its state: the same candidates into the same
            // keys, which a minimum does not notice
            const int mb_first = PACK ? sb << lgR : sb, mb_last = PACK ? imin(mb_first + (1 << lgR) - 1, nmb - 1) : sb;
            const int mb = PACK ? imin(mb_first + slot, mb_last) : sb;
            // streaming range: every unit count some block of the item pairs with inside the target group
            const int mlo = imax(yM0, a_g0 - (qM0 + 8 * mb_last + 7)), mhi = imin(yM1, a_g1 - (qM0 + 8 * mb_first));
            if (mlo > mhi) return;
            double bb2[8], bbt[8], btm[8], acc[8];
            const double2 *const pairS = pair + fillY + ql;
            const double *const tmS = tmv + fillY + ql;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (PACK) { // each lane reads its own block's records
                    const int tab = 8 * mb + i;
                    Rec24 rc = load24(src.s, (__umul24(imin(tab, nS - 1), t.tab_recs) + (ql << shS)) * 32u);
                    if (tab >= nS) rc.a.x = rc.a.y = kNone;
                    rc = combine(rc, !y_left);
                    bb2[i] = rc.a.x; bbt[i] = rc.a.y; btm[i] = rc.tm;
                } else {
                    const double2 p = pairS[i * 8];
                    bb2[i] = p.x; bbt[i] = p.y; btm[i] = tmS[i * 8];
                }
                acc[i] = kNone;
            }
            const int j0 = (mlo - mhi - 1) & 7;
            int mbase = mlo - j0; // step j of a group handles streaming unit count mbase + j; the first group may start at j0
            // row of the key table of target y + q0.  Minima of targets outside the group are dropped: in the plain
            // variant those of the first steps (rows below 0) and of the drain, side by side by lane.
            int row = mbase + qM0 + 8 * mb - a_g0;
            unsigned long long *kcol = s_acc + (PACK ? col : row * 64 + col);
            // one step: the streaming record y against the eight stationary ones, candidates for the
            // targets y + q0 + i, into the rotating minima; then the minimum of target y + q0 is
            // complete for this item.  The streaming record of the NEXT step is read before this
            // step's atomic, so that its latency hides behind the arithmetic (LDS operations
            // complete in order, and the compiler may not move a read over an atomic).
            const double2 *pa = pair + (mlo - yM0) * 8 + yl; // streaming record of the next step
            const double *ta = tmv + (mlo - yM0) * 8 + yl;
            double2 p = *pa;
            double atm = *ta;
            auto merge = [&](int j, const double T) {
                if (PACK ? (unsigned)(row + j) < (unsigned)na : row + j >= 0)
                    atomicMin(PACK ? kcol + (row + j) * 64 : kcol + j * 64, (unsigned long long)__double_as_longlong(fma(T, KS, kd)));
            };
#define OOB_STEP(j)                                                                                   \
    {                                                                                                 \
        pa += 8; ta += 8;                                                                             \
        const double2 pn = *pa; /* may read one record past the last one: staged memory, unused */    \
        const double tn = *ta;                                                                        \
        /* the eighth candidate is the first one of its target: its slot was flushed one step ago */  \
        four_candidates<false>(acc[(j) & 7], acc[((j) + 1) & 7], acc[((j) + 2) & 7], acc[((j) + 3) & 7], bb2, bbt, btm, p, atm); \
        four_candidates<true>(acc[((j) + 4) & 7], acc[((j) + 5) & 7], acc[((j) + 6) & 7], acc[((j) + 7) & 7], bb2 + 4, bbt + 4, btm + 4, p, atm); \
        merge(j, acc[(j)]);                                                                           \
        p = pn; atm = tn;                                                                             \
    }
            if (j0) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j >= j0) OOB_STEP(j)
                mbase += 8; row += 8;
                if (!PACK) kcol += 8 * 64;
            }
            for (; mbase <= mhi; mbase += 8) {
#pragma unroll
                for (int j = 0; j < 8; ++j) OOB_STEP(j)
                row += 8;
                if (!PACK) kcol += 8 * 64;
            }
#undef OOB_STEP
            // the last step was j = 7 with unit count mhi: minima 0..6 belong to targets mhi + q0 + 1 + i
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                if (!PACK && row + i >= na) break;
                merge(i, acc[i]);
            }
        };
        if (lgR > 0) {
            int slot, ue, ve; // this lane's block among the item's, its row and column
            if (lr <= lc) {   // rows 0..2^lr-1, all columns
                slot = lane >> (3 + lr); ue = (lane >> 3) & ((1 << lr) - 1); ve = lane & 7;
            } else {          // all rows, the last 2^lc columns
                const int w = lane & ((8 << lc) - 1);
                slot = lane >> (3 + lc); ue = w >> lc; ve = 8 - (1 << lc) + (w & ((1 << lc) - 1));
            }
            for (int item = 0; item < nsup; ++item) run(std::true_type{}, item, slot, ue, ve);
            preS = loadS(next, 0);
        } else {
            for (int item = 0; item < nmb; ++item) {
                if (item == nmb - 1 && lt > last) preS = Rec24{make_double2(kNone, kNone), 0.0};
                store(fillY + lane, combine(preS, !y_left));
                preS = item + 1 < nmb ? loadS(src, item + 1) : loadS(next, 0); // in flight during this item
                wave_fence();
                run(std::false_type{}, item, 0, lane >> 3, lane & 7);
                wave_fence();
            }
        }
        wave_fence();
    }
    wg_sync();
    // merge into the level's keys, total, split and split point: other splits and segments of the same block do the
    // same
    const int kb = key_bits(L);
    unsigned long long *const dst = t.key + ((long long)(fam_base + a_g0 - ka.dlo) * ka.NT + tile) * 64;
    const long long row = (long long)ka.NT * 64; // keys of one device set
    for (int e = threadIdx.x; e < na * 64; e += blockDim.x) {
        const unsigned long long part = s_acc[e];
        if (part == kNoneBits) continue;
        const unsigned long long key = wide_key(__longlong_as_double((long long)part), s, kb);
        atomicMin(dst + (e >> 6) * row + (e & 63), key);
    }
}

// Per level: the list of (block, segment) workgroup tasks, written once per call.
// by_row = 0 (default): blocks by decreasing distance from the diagonal, the longest split ranges
// first.  by_row = 1 (handle option OOB_OPT_XCD_ORDER, used together with xcd_chunked): block row ub, then segment,
// then the blocks of that row from the far end, so that neighbours in the list split at the same
// points k and stage the same left-child records.
// Bound by the longest list (819 tasks at 98 layers, level 2), hence a task per thread in the default order: one thread for
// a level's list made the set-up launch 56 instead of 17 us, headline workload 7.59 -> 7.49 ms, 61 layers host to host 1.339 -> 1.332 ms.
__device__ void seg_tab_body(const Tables &t, int S, int by_row) {
    if (S > t.sh.Smax) return;
    const int L = t.sh.L, NB = nblocks_of(L), ubmax = (L - S) / 8, dmin = tile_dmin(L, S), target = seg_target(L, S);
    int2 *out = t.seg_tab + (long long)(S - 2) * t.seg_stride;
    auto task = [](int tile, int ub, int vb, int kr, int c, int j) {
        int ofs, len;
        seg_span(kr, c, j, &ofs, &len);
        return make_int2(tile | len << 16, ub | vb << 8 | ofs << 16);
    };
    int n = 0;
    if (!by_row) { // diagonal after diagonal, the tasks of one side by side: its blocks have equally many segments
        int tt = 0;
        for (int d = NB - 1; d >= dmin; --d) {
            const int blocks = imin(ubmax, NB - 1 - d) + 1, kr = tile_krange(L, S, 0, d), c = seg_n(kr, target);
            for (int e = threadIdx.x; e < blocks * c; e += blockDim.x) {
                const int u = e / c;
                out[n + e] = task(tt + u, u, u + d, kr, c, e - u * c);
            }
            n += blocks * c;
            tt += blocks;
        }
        return;
    }
    if (threadIdx.x != 0) return;
    for (int u = 0; u <= imin(ubmax, NB - 1 - dmin); ++u) {
        const int cmax = seg_n(tile_krange(L, S, u, NB - 1), target); // the row's longest split range
        for (int j = 0; j < cmax; ++j) {
            int tt = u; // index of block (u, u + d) in tile order: the blocks of all larger d come first
            for (int d = NB - 1; d >= dmin; --d) {
                if (u + d <= NB - 1 && j < seg_n(tile_krange(L, S, u, u + d), target))
                    out[n++] = task(tt, u, u + d, tile_krange(L, S, u, u + d), seg_n(tile_krange(L, S, u, u + d), target), j);
                tt += imin(ubmax, NB - 1 - d) + 1;
            }
        }
    }
}

// Everything up to level 1, as one launch of kSetupThreads-wide workgroups: workgroup 0 the set-up, `ones` workgroups
// level 1, Smax-1 the task lists of the levels 2 .. Smax, the rest set the n keys of either buffer to "no such state".
// The four parts touch disjoint memory.
__global__ void __launch_bounds__(kSetupThreads) k_prepare(Tables t, oob_profile prof, int how, int by_row, int ones,
                                                           long long stride, long long n) {
    const int nseg = imax(t.sh.Smax - 1, 0);
    int b = blockIdx.x;
    if (b == 0) { setup_body(t, prof, how); return; }
    if (b <= ones) { level1_body(t, prof, b - 1); return; }
    b -= ones;
    if (b <= nseg) { seg_tab_body(t, b + 1, by_row); return; }
    const long long i = (long long)(b - 1 - nseg) * blockDim.x + threadIdx.x;
    if (i < 2 * n) t.key[i < n ? i : stride + i - n] = kNoKey;
}

// ---------------------------------------------------------------------------------------
// Levels S' >= 2, second kernel: grid (block of the plane, delta), one lane per state.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ Rec24 load24(const Rec *p) { return load24(p, 0); }
// Eq. 1-3 for one candidate from the (T, T1, tmax) of its children.
__device__ __forceinline__ double cand_total(const Rec24 &a, const Rec24 &b, double cl, double cr) {
    return a.tm >= b.tm ? (a.a.x + cl * a.tm) + 2.0 * b.a.y : a.a.y + (b.a.x + cr * b.tm);
}

// A state's record: from the candidate that gives it (Eq. 1, 3), or "no such state".
__device__ __forceinline__ void write_state(const Tables &t, long long at, bool exists, double T, double T1, double tmax, int choice) {
    t.rec[at] = exists ? Rec{T, T1, tmax, choice} : Rec{kNone, kNone, 0.0, 0};
}

// Without the keys of k_split_key: the per-split minima of k_split (flags[1]), or every candidate.
constexpr int kSelPairs = 2; // pairs of child records a lane has in flight while it looks for the first m
__device__ void select_lane_per_state(const Tables &t, int Sp, int NT, int NAall) {
    const int L = t.sh.L, M = t.sh.M, lane = threadIdx.x;
    const long long trecs = t.tab_recs;
    int ub, vb;
    tile_decode(L, Sp, blockIdx.x, &ub, &vb);
    const int aidx = blockIdx.y, delta = dlo_of(Sp, M) + aidx;
    const int u = ub * 8 + (lane >> 3), v = vb * 8 + (lane & 7) - t.coff;
    double best = kNone, T1 = kNone, tmax = 0.0;
    int bs = 0, bk = 0;
    if (t.flags[1]) {
        for (int s = 1; s < Sp; ++s) { // first s with the smallest minimum
            const long long o = (((long long)(s - 1) * NAall + aidx) * NT + blockIdx.x) * 64 + lane;
            const double T = t.partT[o];
            if (T < best) { best = T; bs = s; bk = t.partK[o]; }
        }
    }
    const Family fam = family_of(delta, M);
    int bm = 0;
    if (!t.flags[1]) {
        // Totals too large for keys (decided by the set-up kernel from the profile): every candidate
        // (s, k, m) of this state in that order with a strict-minimum update.  Slow, exact, rare.
        if (v <= L && v - u >= Sp)
            for (int s = 1; s < Sp; ++s) {
                const int r = Sp - s;
                int mlo, mhi;
                m_range(fam.fam, fam.units, s, r, M, t.sh.n_max, &mlo, &mhi);
                const double cl = t.sh.Nb > 0 ? -(double)r : 3.0 * r, cr = t.sh.Nb > 0 ? 0.0 : 4.0 * s;
                const Rec *baseA = t.rec + (level(t, s).base + fam.fam_base) * trecs;
                const Rec *baseB = t.rec + (level(t, r).base + fam.fam_base + fam.units) * trecs;
                for (int k = u + s; k <= v - r; ++k) {
                    const Rec *atA = baseA + rec_off(u, k, t.coff, t.NB), *atB = baseB + rec_off(k, v, t.coff, t.NB);
                    for (int m = mlo; m <= mhi; ++m) {
                        const Rec24 a = load24(atA + m * trecs), b = load24(atB - m * trecs);
                        const double T = cand_total(a, b, cl, cr);
                        if (T < best) { best = T; bs = s; bk = k; bm = m; T1 = a.a.y + b.a.y; tmax = fmax(a.tm, b.tm); }
                    }
                }
            }
    } else if (best < kNone) {
        const int r = Sp - bs;
        int mlo, mhi;
        m_range(fam.fam, fam.units, bs, r, M, t.sh.n_max, &mlo, &mhi);
        const double cl = t.sh.Nb > 0 ? -(double)r : 3.0 * r, cr = t.sh.Nb > 0 ? 0.0 : 4.0 * bs;
        // first m whose candidate equals the minimum; kSelPairs candidates' records in flight at a time
        const Rec *atA = t.rec + (long long)(level(t, bs).base + fam.fam_base) * trecs + rec_off(u, bk, t.coff, t.NB);
        const Rec *atB = t.rec + (long long)(level(t, r).base + fam.fam_base + fam.units) * trecs + rec_off(bk, v, t.coff, t.NB);
        for (int m0 = mlo; m0 <= mhi && bm == 0; m0 += kSelPairs) {
            Rec24 ra[kSelPairs], rb[kSelPairs];
#pragma unroll
            for (int q = 0; q < kSelPairs; ++q) {
                const int m = imin(m0 + q, mhi);
                ra[q] = load24(atA + m * trecs);
                rb[q] = load24(atB - m * trecs);
            }
#pragma unroll
            for (int q = 0; q < kSelPairs; ++q)
                if (bm == 0 && m0 + q <= mhi && cand_total(ra[q], rb[q], cl, cr) == best) {
                    bm = m0 + q; T1 = ra[q].a.y + rb[q].a.y; tmax = fmax(ra[q].tm, rb[q].tm);
                }
        }
    }
    if (best < kNone && bm == 0) *t.status = kInternalError;
    write_state(t, rec_block(t, Sp, delta, ub, vb) + lane, best < kNone && bm, best, T1, tmax, bs | bk << 10 | bm << 21);
}
__global__ void __launch_bounds__(64) k_select(Tables t, int Sp, int NT, int NAall) {
    select_lane_per_state(t, Sp, NT, NAall);
}

// ---------------------------------------------------------------------------------------
// Levels S' >= 2, second kernel, keyed path: grid (block of the plane, delta, LPS parts of the block),
// LPS lanes per state.
//
// The lanes of a state share out what the state has to look at, so that each dependent round trip
// to memory covers LPS times as much as it would with one lane per state; the kernel sits on the
// chain between the levels and its duration is made of such round trips.
//   1. FUSE only: the two outer splits s = 1 and s = S'-1, whose one-stage child has a single unit
//      count across nodes (a line of candidates instead of a rectangle), are evaluated here,
//      candidate by candidate from the child records; no split kernel is launched for them.
//   2. The key of the (other) splits holds the smallest (T, s, k).
//   3. FUSE only: the lanes' partial minima are merged in the order (T, s, k, m).
//   4. A winner that came from a key does not know its m yet: the lanes test LPS m at a time.
//   5. The lane that has seen the winner forms the record from the two child records it has read.
// Without keys (flags[0] = 0) the wave of part 0 evaluates the block one lane per state as k_select does.
// ---------------------------------------------------------------------------------------
constexpr int kSel8Outer = 4;  // candidates of the outer splits a lane has in flight
constexpr int kSel8M = 2;      // m a lane tests per round

template <int LPS, bool FUSE>
__global__ void __launch_bounds__(64) k_select_key(Tables t, int Sp, int NT, int NAall) {
    if (t.flags[0] == 0) {
        if (blockIdx.z == 0) select_lane_per_state(t, Sp, NT, NAall);
        return;
    }
    const int L = t.sh.L, M = t.sh.M, lane = threadIdx.x, sub = lane & (LPS - 1);
    int ub, vb;
    tile_decode(L, Sp, blockIdx.x, &ub, &vb);
    const int aidx = blockIdx.y, delta = dlo_of(Sp, M) + aidx;
    const int tl = blockIdx.z * (64 / LPS) + lane / LPS, u = ub * 8 + (tl >> 3), v = vb * 8 + (tl & 7) - t.coff;
    const bool valid = v <= L && v - u >= Sp;
    const Family fam = family_of(delta, M);
    const bool fixed_nb = t.sh.Nb > 0;
    const long long trecs = t.tab_recs;
    double best = kNone, T1 = kNone, tmax = 0.0; // (of the candidate this lane has seen for it)
    unsigned btag = 0xffffffffu; // s << 21 | k << 10 | m (m = 0: not known yet)

    if (FUSE && valid) {
        const int nk = v - u - Sp + 1; // split points u + s .. v - r of either outer split
        for (int side = 0; side < (Sp > 2 ? 2 : 1); ++side) {
            const int s = side ? Sp - 1 : 1, r = Sp - s;
            int mlo, mhi;
            m_range(fam.fam, fam.units, s, r, M, t.sh.n_max, &mlo, &mhi);
            const double cl = fixed_nb ? -(double)r : 3.0 * r, cr = fixed_nb ? 0.0 : 4.0 * s;
            const Rec *baseA = t.rec + (level(t, s).base + fam.fam_base) * trecs;
            const Rec *baseB = t.rec + (level(t, r).base + fam.fam_base + fam.units) * trecs;
            for (int m = mlo; m <= mhi; ++m)
                for (int j0 = sub; j0 < nk; j0 += LPS * kSel8Outer) {
                    Rec24 ra[kSel8Outer], rb[kSel8Outer];
                    int kk[kSel8Outer];
#pragma unroll
                    for (int q = 0; q < kSel8Outer; ++q) { // past the end: the last candidate again
                        const int k = u + s + imin(j0 + LPS * q, nk - 1);
                        kk[q] = k;
                        ra[q] = load24(baseA + m * trecs + rec_off(u, k, t.coff, t.NB));
                        rb[q] = load24(baseB - m * trecs + rec_off(k, v, t.coff, t.NB));
                    }
#pragma unroll
                    for (int q = 0; q < kSel8Outer; ++q) {
                        const double T = cand_total(ra[q], rb[q], cl, cr);
                        const unsigned tag = ((unsigned)s << 21) | ((unsigned)kk[q] << 10) | (unsigned)m;
                        if (T < best || (T == best && tag < btag)) {
                            best = T; btag = tag; T1 = ra[q].a.y + rb[q].a.y; tmax = fmax(ra[q].tm, rb[q].tm);
                        }
                    }
                }
        }
    }
    if (valid) { // the consumed key goes back to "no such state"
        const int kb = key_bits(L), mask = (1 << kb) - 1;
        unsigned long long *const at = t.key + ((long long)aidx * NT + blockIdx.x) * 64 + tl;
        const unsigned long long key = *at;
        if (key != kNoKey) {
            const double T = (double)(long long)(key >> 2 * kb);
            const unsigned tag = ((unsigned)(key >> kb) & mask) << 21 | ((unsigned)key & mask) << 10;
            if (T < best || (T == best && tag < btag)) { best = T; btag = tag; }
            if (sub == 0) *at = kNoKey;
        }
    }
    bool mine = sub == 0; // the lane that writes the state's record
    if (FUSE) { // the lanes of a state: smallest (T, s, k, m)
        const unsigned own = btag;
#pragma unroll
        for (int d = 1; d < LPS; d <<= 1) {
            const double ob = __shfl_xor(best, d, 64);
            const unsigned ot = (unsigned)__shfl_xor((int)btag, d, 64);
            if (ob < best || (ob == best && ot < btag)) { best = ob; btag = ot; }
        }
        if ((btag & 1023u) && best < kNone) mine = own == btag; // an outer split: the lane that has seen it (tags are unique)
    }
    const int bs = (int)(btag >> 21), bk = (int)((btag >> 10) & 2047u);
    int bm = (int)(btag & 1023u);
    if (best < kNone && bm == 0) { // first m whose candidate equals the minimum, the lanes side by side
        const int r = Sp - bs;
        int mlo, mhi;
        m_range(fam.fam, fam.units, bs, r, M, t.sh.n_max, &mlo, &mhi);
        const double cl = fixed_nb ? -(double)r : 3.0 * r, cr = fixed_nb ? 0.0 : 4.0 * bs;
        const Rec *baseA = t.rec + (level(t, bs).base + fam.fam_base) * trecs +
                           rec_off(u, bk, t.coff, t.NB);
        const Rec *baseB = t.rec + (level(t, r).base + fam.fam_base + fam.units) * trecs +
                           rec_off(bk, v, t.coff, t.NB);
        for (int m0 = mlo + sub; m0 - sub <= mhi && bm == 0; m0 += LPS * kSel8M) {
            Rec24 ra[kSel8M], rb[kSel8M];
#pragma unroll
            for (int q = 0; q < kSel8M; ++q) {
                const int m = imin(m0 + LPS * q, mhi);
                ra[q] = load24(baseA + m * trecs);
                rb[q] = load24(baseB - m * trecs);
            }
            int found = 0x7fffffff;
#pragma unroll
            for (int q = kSel8M - 1; q >= 0; --q) {
                const int m = m0 + LPS * q;
                if (m <= mhi && cand_total(ra[q], rb[q], cl, cr) == best) { found = m; T1 = ra[q].a.y + rb[q].a.y; tmax = fmax(ra[q].tm, rb[q].tm); }
            }
            int first = found;
#pragma unroll
            for (int d = 1; d < LPS; d <<= 1) first = imin(first, __shfl_xor(first, d, 64));
            if (first != 0x7fffffff) { bm = first; mine = found == first; }
        }
    }
    if (!mine) return;
    if (best < kNone && bm == 0) *t.status = kInternalError;
    write_state(t, rec_block(t, Sp, delta, ub, vb) + tl, best < kNone && bm, best, T1, tmax, bs | bk << 10 | bm << 21);
}

// ---------------------------------------------------------------------------------------
// Levels S' >= 2, small levels: grid (block of the plane, delta, part of the block); one launch does the level.
//
// A level of few candidates is bound by its launches and the chain inside them, so splits and select are
// one kernel without keys: a workgroup evaluates C = 2^lgC neighbouring states (u, v) of a row of a block, candidate by candidate
// from the child records, 256 / C lanes a state.  The lanes of a wave are C columns times 64 / C consecutive split
// points.
// The (s, m) pairs of the device set are listed in LDS first, beside the offsets of the split points' records; candidate i is
// pair i / nk, split point i % nk of the widest state (a narrower one reads "no such state" beyond its own).
// Smallest (T, s, k, m) by comparison, so the kernel does not depend on keys fitting a double.
//
// What bounds it: the workgroup with the most candidates a lane.  With 32 lanes for every state and the records' places formed from
// scratch for each candidate (850 cycles each) the slowest workgroup took 23 000 cycles where the others took 10 000, whatever was in
// flight (8 or 10 candidates a lane: no change); then 13 000 and 10 000, of them 1 100 for the list of pairs and 2 000 for a second look
// at the winner's children, which a state without T3 and k* does not take.  26 layers: 9 -> 6 us a level, 232 -> 176 us a call, without the
// second look 155.
// ---------------------------------------------------------------------------------------
constexpr int kSmallPairs = 1024;  // (s, m) pairs of a device set the kernel has room for
constexpr int kSmallThreads = 256;
constexpr int kSmallFlight = 4;    // candidates a lane has in flight
__global__ void __launch_bounds__(kSmallThreads) k_level_small(Tables t, int Sp, int lgC) {
    __shared__ int4 s_pair[kSmallPairs]; // left table, right table (byte offsets of their first records), s << 21 | m, s
    __shared__ int2 s_off[OOB_MAX_L + 1]; // split point u + i: byte offset of left record (u, u + i), of row u + i of the right records
    __shared__ unsigned long long s_best[8];
    __shared__ unsigned s_tag[8];
    const int L = t.sh.L, M = t.sh.M, n_max = t.sh.n_max, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int ub, vb;
    tile_decode(L, Sp, blockIdx.x, &ub, &vb);
    const int delta = dlo_of(Sp, M) + blockIdx.y;
    const Family fam = family_of(delta, M);
    const int row = blockIdx.z >> (3 - lgC), col0 = (blockIdx.z & ((8 >> lgC) - 1)) << lgC, C = 1 << lgC, col = tid & (C - 1);
    const int u = ub * 8 + row, vcol = col0 + col, nk = vb * 8 + col0 + C - 1 - t.coff - u - Sp + 1;
    const long long out_at = (long long)(level(t, Sp).base + delta) * t.tab_recs + tri_index(ub, vb, t.NB) * 64 + (row << 3) + vcol;
    if (nk <= 0) { // no states here
        if (tid >= C) return;
        write_state(t, out_at, false, kNone, kNone, 0.0, 0);
        return;
    }
    const unsigned tab_bytes = (unsigned)t.tab_recs * (unsigned)sizeof(Rec);
    const bool fixed_nb = t.sh.Nb > 0;
    if (tid < 8) { s_best[tid] = kNoKey; s_tag[tid] = 0xffffffffu; }
    for (int i = tid; i < nk + Sp; i += kSmallThreads) { // split points u + 1 .. u + nk + Sp - 2
        const int k = u + i, kb = k >> 3;
        s_off[i] = make_int2(((ub * t.NB - ub * (ub - 1) / 2 - ub + ((k + t.coff) >> 3)) * 64 + ((u & 7) << 3) + ((k + t.coff) & 7)) * (int)sizeof(Rec),
                             ((kb * t.NB - kb * (kb - 1) / 2 + vb - kb) * 64 + ((k & 7) << 3)) * (int)sizeof(Rec));
    }
    int np = 0;
    for (int s0 = 1; s0 < Sp; s0 += 64) { // every wave counts the pairs of 64 splits, each writes a share of them
        const int s = s0 + lane, r = Sp - s;
        int mlo = 1, mhi = 0;
        Level dA = {0, 0}, dB = {0, 0};
        if (r > 0) { // unit counts of the children (child_units with the level's ceil(S / M))
            dA = level(t, s); dB = level(t, r);
            const int alo = fam.fam ? dA.least : s, ahi = fam.fam ? imin(s, n_max) : M - 1;
            const int blo = fam.fam ? dB.least : r, bhi = fam.fam ? imin(r, n_max) : M - 1;
            mlo = imax(alo, fam.units - bhi);
            mhi = imin(ahi, fam.units - blo);
        }
        const int cnt = imax(0, mhi - mlo + 1), incl = scan_int(cnt), at = np + incl - cnt;
        for (int m = mlo + wave; m <= mhi; m += kSmallThreads / 64)
            if (at + m - mlo < kSmallPairs) // (the host has checked that they fit)
                s_pair[at + m - mlo] = make_int4((dA.base + fam.fam_base + m) * tab_bytes, (dB.base + fam.fam_base + fam.units - m) * tab_bytes, s << 21 | m, s);
        np += __builtin_amdgcn_readlane(incl, 63);
    }
    np = imin(np, kSmallPairs);
    wg_sync();
    double best = kNone, T1 = kNone, tmax = 0.0;
    unsigned btag = 0xffffffffu; // s << 21 | k << 10 | m
    const int total = np * nk, g = tid >> lgC;
    if (np > 0) {
        const int G = kSmallThreads >> lgC, dp = G / nk, dk = G - dp * nk;
        const char *const rec = (const char *)t.rec;
        const unsigned right = (unsigned)vcol * (unsigned)sizeof(Rec);
        int p = g / nk, kk = g - p * nk;
        for (int i = g; i < total; i += G * kSmallFlight) {
            Rec24 ra[kSmallFlight], rb[kSmallFlight];
            unsigned tag[kSmallFlight];
#pragma unroll
            for (int q = 0; q < kSmallFlight; ++q) {
                const int4 e = s_pair[imin(p, np - 1)]; // past the end: some candidate of the last pair again
                const int2 o = s_off[e.w + kk];
                ra[q] = load24(rec, (unsigned)e.x + (unsigned)o.x);
                rb[q] = load24(rec, (unsigned)e.y + (unsigned)o.y + right);
                tag[q] = (unsigned)e.z + ((unsigned)(u + e.w + kk) << 10);
                p += dp; kk += dk;
                if (kk >= nk) { kk -= nk; ++p; }
            }
#pragma unroll
            for (int q = 0; q < kSmallFlight; ++q) {
                const int s = (int)(tag[q] >> 21), r = Sp - s;
                const double T = cand_total(ra[q], rb[q], fixed_nb ? -(double)r : 3.0 * r, fixed_nb ? 0.0 : 4.0 * s);
                if (T < best || (T == best && tag[q] < btag)) { best = T; btag = tag[q]; T1 = ra[q].a.y + rb[q].a.y; tmax = fmax(ra[q].tm, rb[q].tm); }
            }
        }
    }
    // the state's smallest total (as integers: non-negative doubles), then the smallest tag among those that have it; the lane
    // that has both writes the record
    const unsigned long long mine = (unsigned long long)__double_as_longlong(best);
    if (best < kNone) atomicMin(&s_best[col], mine);
    wg_sync();
    const unsigned long long least = s_best[col];
    if (mine == least) atomicMin(&s_tag[col], btag);
    wg_sync();
    if (mine != least || s_tag[col] != btag || (least == kNoKey && g > 0)) return;
    const int s = (int)(btag >> 21), k = (int)((btag >> 10) & 2047u), m = (int)(btag & 1023u);
    write_state(t, out_at, best < kNone, best, T1, tmax, s | (k << 10) | (m << 21));
}

// ---------------------------------------------------------------------------------------
// Template extraction ("Choosing the number of stages"): one wave per template size
// n = n_min + blockIdx.x, the lanes share out the stage counts; smallest T, then smallest S.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_pick(Tables t, oob_templates out) {
    const int i = blockIdx.x, lane = threadIdx.x;
    const int L = t.sh.L, M = t.sh.M, n = t.sh.n_min + i, delta = M - 2 + n;
    double best = kNone;
    int bestS = 0x7fffffff;
    if (n <= t.sh.n_max)
        for (int S = n + lane; S <= t.sh.Smax; S += 64) { // ascending per lane: the first minimum stays
            if (delta < dlo_of(S, M) || delta > dhi_of(S, M, t.sh.n_max)) continue;
            const double T = t.rec[rec_index(t, S, delta, 0, L)].T;
            if (T < best) { best = T; bestS = S; }
        }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double ob = __shfl_xor(best, d, 64);
        const int os = __shfl_xor(bestS, d, 64);
        if (ob < best || (ob == best && os < bestS)) { best = ob; bestS = os; }
    }
    if (lane != 0) return;
    if (!(best < kNone)) bestS = 0;
    out.feasible[i] = bestS > 0;
    out.S[i] = bestS;
    long long T = 0, T1 = 0, tm = 0;
    if (bestS > 0) {
        const Rec r = t.rec[rec_index(t, bestS, delta, 0, L)];
        T = (long long)best; T1 = (long long)r.T1; tm = (long long)r.tmax;
    }
    out.T[i] = T; out.T1[i] = T1; out.tmax[i] = tm;
    out.T2[i] = out.T3[i] = out.kstar[i] = 0; // k_backtrack, where there is a pipeline
}

// ---------------------------------------------------------------------------------------
// Node specification and coverage (Section 4.1.1, Appendix A), one workgroup.  The template sizes
// are the consecutive integers n0..n_hi, so c pipelines can use exactly the node counts
// c n0 .. c n_hi; the largest pipeline count whose sizes sum to x is therefore
// c = floor(x / n0) when x <= c n_hi, and x is no sum of sizes at all otherwise (fewer
// pipelines reach even less).  That is the value the coin-change recursion of Section 4.2.1
// gives, without the table.
// ---------------------------------------------------------------------------------------
__device__ void coverage_body(const Tables &t, const oob_templates &out, int len) {
    __shared__ int s_i0, s_i1, s_thm, s_tail;
    const int cnt = t.sh.count, f = t.sh.f, lane = threadIdx.x;
    if (lane == 0) {
        int i0 = -1;
        for (int q = 0; q < cnt; ++q) if (out.feasible[q]) { i0 = q; break; }
        int i1 = i0;
        while (i0 >= 0 && i1 + 1 < cnt && out.feasible[i1 + 1]) ++i1;
        s_i0 = i0; s_i1 = i1; s_thm = 1; s_tail = 1;
    }
    for (int q = lane; q < len; q += blockDim.x) out.cover_maxpipes[q] = 0;
    __syncthreads();
    if (s_i0 < 0) {
        if (lane < 8) out.cover_hdr[lane] = 0;
        return;
    }
    const int n0 = t.sh.n_min + s_i0, n_hi = t.sh.n_min + s_i1, p = n_hi - n0 + 1;
    const int N = n_hi + f * n0;
    const int lo_thm = (f + 1) * n0, lo_tail = N - f < 1 ? 1 : N - f;
    const int lo = lo_thm < lo_tail ? lo_thm : lo_tail;
    for (int x = lo + lane; x <= N; x += blockDim.x) {
        int c = x / n0;
        if ((long long)c * n_hi < x) c = 0;
        if (x - lo < len) out.cover_maxpipes[x - lo] = c;
        if (x >= lo_thm && c < f + 1) atomicMin(&s_thm, 0);
        if (x >= lo_tail && c < 1) atomicMin(&s_tail, 0);
    }
    __syncthreads();
    if (lane == 0) {
        out.cover_hdr[0] = n0; out.cover_hdr[1] = n_hi; out.cover_hdr[2] = p; out.cover_hdr[3] = N;
        out.cover_hdr[4] = p > n0 - 1; out.cover_hdr[5] = lo; out.cover_hdr[6] = s_thm; out.cover_hdr[7] = s_tail;
    }
}

// Stages of each template from the stored (s, k, m) tree: one workgroup per template, one thread
// per stage.  Thread p walks from the root to the p-th leaf (left subtree if p is below the left
// child's stage count, else right with p reduced by it), so the walks of a template run side by
// side and the kernel takes as long as the deepest leaf, not as the whole tree.
// The first slowest stage is k*, the stages from it on make T3 (Eq. 3), k* and tmax make T2 (Eq. 2).
// Workgroup `count` writes the end of the offsets and the coverage.
__global__ void __launch_bounds__(128) k_backtrack(Tables t, oob_templates out, int len) {
    __shared__ int s_part[128];
    __shared__ long long s_time[OOB_MAX_L];
    __shared__ unsigned long long s_T3;
    __shared__ int s_kstar;
    const int i = blockIdx.x, tid = threadIdx.x, cnt = t.sh.count;
    int part = 0;
    for (int q = tid; q < i && q < cnt; q += blockDim.x) part += out.S[q];
    s_part[tid] = part;
    __syncthreads();
    int off = 0;
    for (int q = 0; q < (int)blockDim.x; ++q) off += s_part[q];
    if (tid == 0) out.stage_off[i] = off;
    if (i >= cnt) { coverage_body(t, out, len); return; }
    const int S = out.S[i];
    if (S == 0) return;
    const int L = t.sh.L, M = t.sh.M;
    int *begin = out.stage_begin + off + i, *gpus = out.stage_gpus + off;
    for (int p = tid; p < S; p += blockDim.x) {
        int Sq = S, delta = M - 2 + t.sh.n_min + i, u = 0, v = L, pos = p;
        while (Sq > 1) {
            const int ch = (int)t.rec[rec_index(t, Sq, delta, u, v)].choice;
            const int s = ch & 1023, k = (ch >> 10) & 2047, m = (ch >> 21) & 1023;
            const Family fam = family_of(delta, M);
            if (s < 1 || s >= Sq) { *t.status = kInternalError; break; }
            if (pos < s) { Sq = s; delta = fam.fam_base + m; v = k; }
            else         { pos -= s; Sq -= s; delta = fam.fam_base + fam.units - m; u = k; }
        }
        begin[p] = u;
        gpus[p] = delta < M - 1 ? delta + 1 : M;
        s_time[p] = (long long)t.rec[rec_index(t, Sq, delta, u, v)].T1;
    }
    if (tid == 0) { begin[S] = L; s_kstar = S; s_T3 = 0; }
    __syncthreads();
    const long long tmax = out.tmax[i];
    for (int p = tid; p < S; p += blockDim.x) if (s_time[p] == tmax) { atomicMin(&s_kstar, p); break; } // (a thread's ascend)
    __syncthreads();
    const int ks = s_kstar;
    unsigned long long part3 = 0;
    for (int p = tid; p < S; p += blockDim.x) if (p >= ks) part3 += (unsigned long long)s_time[p];
    if (part3) atomicAdd(&s_T3, part3);
    __syncthreads();
    if (tid == 0) {
        if (ks == S) *t.status = kInternalError;
        const long long nb = t.sh.Nb > 0 ? t.sh.Nb : 4LL * S;
        out.T3[i] = (long long)s_T3;
        out.kstar[i] = ks;
        out.T2[i] = (nb - S + ks - 1) * tmax;
    }
}

// Copies one table into dense n x n arrays, n = L-S'+1, entry [u][v - S'] (tests only).  T3 and k* of a state: down the tree to its
// first slowest stage (Eq. 3).
__global__ void k_export(Tables t, int S, int delta, double *T, double *T1, double *tmax, double *T3,
                         int *kstar, int *choice) {
    const int n = t.sh.L - S + 1;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n * n) return;
    const int u = idx / n, j = idx % n, v = j + S;
    Rec r = {kNone, kNone, 0.0, 0};
    if (j >= u) r = t.rec[rec_index(t, S, delta, u, v)];
    double after = 0.0; // T3
    int ks = 0;
    T[idx] = r.T; T1[idx] = r.T1; tmax[idx] = r.tmax; choice[idx] = (int)r.choice;
    if (r.T < kNone) {
        int Sq = S, d = delta, a = u, b = v;
        Rec x = r;
        while (Sq > 1) {
            const int s = (int)x.choice & 1023, k = ((int)x.choice >> 10) & 2047, m = ((int)x.choice >> 21) & 1023;
            const Family fam = family_of(d, t.sh.M);
            if (s < 1 || s >= Sq) break; // (never: a state's split has stages on both sides)
            const Rec left = t.rec[rec_index(t, s, fam.fam_base + m, a, k)], right = t.rec[rec_index(t, Sq - s, fam.fam_base + fam.units - m, k, b)];
            if (left.tmax >= right.tmax) { after += right.T1; Sq = s; d = fam.fam_base + m; b = k; x = left; }
            else { ks += s; Sq -= s; d = fam.fam_base + fam.units - m; a = k; x = right; }
        }
        after += x.T1;
    }
    T3[idx] = after; kstar[idx] = ks;
}

// ---------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------
inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

long long table_count(int L, int M, int n_max, int Nb) {
    const int Smax = smax_of(L, n_max, M, Nb);
    long long e = 0;
    for (int S = 1; S <= Smax; ++S) {
        const int nd = dhi_of(S, M, n_max) - dlo_of(S, M) + 1;
        if (nd > 0) e += nd;
    }
    return e;
}

// Largest (S'-1) * deltas * tiles over the levels: slots of the per-split minima.
long long part_slots(int L, int M, int n_max, int Nb) {
    const int Smax = smax_of(L, n_max, M, Nb);
    long long best = 1;
    for (int S = 2; S <= Smax; ++S) {
        const long long nd = dhi_of(S, M, n_max) - dlo_of(S, M) + 1;
        if (nd <= 0) continue;
        const long long sl = (long long)(S - 1) * nd * tile_count_bound(L, S);
        if (sl > best) best = sl;
    }
    return best;
}

struct Carve {
    size_t rec, partT, partK, flags, seg_tab, total;
    long long recs, slots;
};
// Byte offsets of the workspace arrays, sized for the handle's maxima.
Carve carve(int L, int nodes, int M) {
    Carve c;
    c.recs = table_count(L, M, nodes, 0) * tri_blocks(nblocks_of(L)) * 64;
    c.slots = part_slots(L, M, nodes, 0);
    const size_t E = (size_t)c.recs;
    const int Smax = smax_of(L, nodes, M, 0);
    size_t o = 0;
    c.rec = o;     o = align_up(o + sizeof(Rec) * E);
    // two buffers of minima: consecutive levels are evaluated side by side (see oob_plan_templates)
    c.partT = o;   o = align_up(o + 2 * sizeof(double) * (size_t)c.slots * 64);
    c.partK = o;   o = align_up(o + sizeof(int) * (size_t)c.slots * 64); // plain kernel only: one stream
    c.flags = o;   o = align_up(o + sizeof(int) * 64);
    // the task list of a level is longest at S' = 2; every level gets that many entries
    c.seg_tab = o; o = align_up(o + sizeof(int2) * ((size_t)imax(Smax - 1, 1) * seg_count_bound(L) + 1));
    c.total = o;
    return c;
}

// Structural work counts of a level: states = (u, v) with v - u >= S' per table; candidates = (s, k, m)
// with both children valid: per (s, m) pair one per (u, k, v), u + s <= k <= v - r.
// *most: (s, m) pairs of the target that has most of them.
// The pairs of a split as a function of the target's units are a trapezoid, two intervals added up: its four corners go into
// second differences, summed twice at the end of the level.  Counted target by target and split by split it took the
// host 960 us before the first launch of the headline workload and 175 us for 61 layers, 27 and 12 us like this: a call at a time
// 7.40 -> 6.78 ms, and 1.33 -> 1.22 ms from host to host.
void level_counts(const Shape &sh, int S, long long *states, long long *cands, int *most) {
    const long long n = sh.L - S + 1;
    const int dlo = dlo_of(S, sh.M), dhi = dhi_of(S, sh.M, sh.n_max);
    long long pairs = 0;
    *most = 0;
    for (int fam = S <= sh.M ? 0 : 1; fam < 2; ++fam) {
        int t_lo, t_hi;
        target_units(fam, S, sh.M, sh.n_max, &t_lo, &t_hi);
        int corner[OOB_MAX_NODES + 1];
        std::fill(corner, corner + imax(0, t_hi - t_lo + 1), 0);
        auto add = [&](int units, int x) { if (units <= t_hi) corner[units - t_lo] += x; }; // (no child pair adds up to less than t_lo)
        for (int s = 1; s < S; ++s) {
            int alo, ahi, blo, bhi;
            child_units(fam, s, sh.M, sh.n_max, &alo, &ahi);
            child_units(fam, S - s, sh.M, sh.n_max, &blo, &bhi);
            if (alo > ahi || blo > bhi) continue;
            add(alo + blo, 1); add(ahi + 1 + blo, -1); add(alo + bhi + 1, -1); add(ahi + bhi + 2, 1);
        }
        for (int units = t_lo, slope = 0, here = 0; units <= t_hi; ++units) {
            slope += corner[units - t_lo];
            here += slope;
            pairs += here;
            *most = imax(*most, here);
        }
    }
    *states = dhi >= dlo ? (dhi - dlo + 1) * (n * (n + 1) / 2) : 0;
    *cands = pairs * (n * (n + 1) * (n + 2) / 6);
}

constexpr size_t kLdsLimit = 160 * 1024; // gfx950: 160 KB of LDS per workgroup
constexpr size_t kLdsPrefer = 64 * 1024; // at least two workgroups per compute unit

// Launch shape of k_split for one family of one level.
struct SplitPlan { int waves, groups, pc, ntab, na, cap, full, range; size_t lds; }; // (cap, full, range: k_split_key)
bool plan_split(const Shape &sh, int Sp, int fam, SplitPlan *p) {
    int t_lo, t_hi;
    target_units(fam, Sp, sh.M, sh.n_max, &t_lo, &t_hi);
    if (fam == 0 && Sp > sh.M) return false;
    if (t_hi < t_lo) return false;
    const int cnt = t_hi - t_lo + 1;
    p->waves = imin(8, cdiv(cnt, 8));
    p->groups = cdiv(cnt, 8 * p->waves);
    int ntab = 1;
    for (int s = 1; s < Sp; ++s) {
        int A_lo, A_hi, B_lo, B_hi;
        child_units(fam, s, sh.M, sh.n_max, &A_lo, &A_hi);
        child_units(fam, Sp - s, sh.M, sh.n_max, &B_lo, &B_hi);
        for (int g = 0; g < p->groups; ++g) {
            const int a0 = t_lo + g * p->waves * 8, a1 = imin(t_hi, a0 + p->waves * 8 - 1);
            const int mA0 = imax(A_lo, a0 - B_hi), mA1 = imin(A_hi, a1 - B_lo);
            const int mB0 = imax(B_lo, a0 - A_hi), mB1 = imin(B_hi, a1 - A_lo);
            if (mA0 <= mA1 && mB0 <= mB1) ntab = imax(ntab, mA1 - mA0 + 1 + mB1 - mB0 + 1 + 1);
        }
    }
    const size_t per_k = (size_t)ntab * 8 * 24;
    p->pc = per_k * 4 <= kLdsPrefer ? 4 : per_k * 2 <= kLdsPrefer ? 2 : 1;
    p->lds = per_k * p->pc;
    return true;
}

int env_or(const char *name, int dflt) {
    const char *v = getenv(name);
    return v && *v ? atoi(v) : dflt;
}
// Debug knobs, read once when the library is loaded (the defaults are the measured optimum).
static const int kKeyWaves = imin(env_or("OOB_TUNE_KEY_WAVES", 4), 4);
static const int kKeyPack = env_or("OOB_TUNE_KEY_PACK", 1);
static const int kBatchOverlap = env_or("OOB_TUNE_BATCH_OVERLAP", 0);
static const int kBatchLanes = env_or("OOB_TUNE_BATCH_LANES", 8);
// From this level on the select kernel works with eight lanes per state and evaluates the two outer
// splits itself (below it the machine is full of split workgroups, and eight times the waves of
// the plain select only wait longer for a place); measured on the headline workload, where 78-88 gave
// the same time.  Handle options move both thresholds.
constexpr int kSelect8From = 82, kFuseFrom = 82;
// Levels that k_level_small does: as many candidates of the widest state as 32 lanes look at in five round trips, and
// so few in all that their scattered reads are not what the launch takes (it reads 0.15 million candidates a
// microsecond).  Measured against split and select launches, with eight columns a workgroup: 26 layers 308 -> 232 us with the line at 640
// (320: 274 us, 1 000: 232 us), smallest job 39 -> 27 us on the GPU; 61 layers 1 294 us either way (1 000: 1 315 us).
// A million candidates of the level instead of half a million: 48 layers x 8 GPUs x 8 nodes 497 instead of 473 us, 75 x 4 x 10 384 instead of 391.
constexpr int kSmallState = 640, kSmallLevel = 500000;
// Columns of a workgroup (lgC) of such a level whose widest state has `most` candidates: eight, or fewer as long as a lane then has more
// than kSmallSerial of them one after the other and the launch no more than kSmallGroups workgroups.  A candidate is some
// hundred cycles of a wave that is alone on its SIMD, and the workgroup of the widest state with the most of them is what a launch waits for.  (All
// with the second look at the winner's children, which is the same for every line.)  26 layers, kSmallSerial, kSmallGroups: 4, 2 048 176 us; 4, 1 024 174; 8, 1 024 176; 2, 2 048 182; 4, 4 096 187; eight columns always 232.
// 31 jobs of 12 to 98 layers drawn at random, against 4, 2 048 (geometric mean, best, worst): 4, 1 024 1.01, 0.94, 1.05; 8, 2 048 1.03, 0.92, 1.11; 2, 2 048
// 1.03, 0.95, 1.13; 4, 4 096 1.03, 0.94, 1.25; eight columns always 1.05, 0.93, 1.20.
constexpr int kSmallSerial = 4, kSmallGroups = 2048;
static int small_columns(const Shape &sh, int S, long long most) {
    const long long groups = (long long)tile_count(sh.L, S) * (dhi_of(S, sh.M, sh.n_max) - dlo_of(S, sh.M) + 1) * 8;
    int lgC = 3;
    while (lgC > 0 && most > (long long)kSmallSerial * (kSmallThreads >> lgC) && groups << (4 - lgC) <= kSmallGroups) --lgC;
    return lgC;
}
// So do levels on one stream of a job that has the GPU to itself, where a state has more than kSel8Range m to look through for some split and
// eight lanes a state still find a place at once: 61 layers 1 181 -> 1 124 us with it from level 20 on, 1 144 from level 8 on (short ranges); beside the
// other jobs of a batch or the inner splits of the next level the waves wait for a place instead (batch of 32 jobs 74.8 -> 80 ms).  488 jobs of 12 to 160
// layers, 2 to 64 nodes of 1, 2, 4 and 8 GPUs, against one lane a state: 0.95 to 1.00 of the time where it applies (a single job with one_stream set has no such level).
constexpr int kSel8Range = 8, kSel8Waves = 8192;
constexpr int kOverlapFrom = 24000; // thousand candidates of a level: see enqueue_job
constexpr int kSelLanes = 1; // lanes per state below that
// Waves of k_split_key on a compute unit in workgroups of w of them, which share the key table.
static int key_waves_on(int na, int ntab, int w) {
    return imin((int)(kLdsLimit / ((size_t)na * 512 + (size_t)w * ntab * 192)) * w, 4 * kWavesPerSimd);
}
// Waves per workgroup of a keyed launch: as many as put the most waves on a compute unit, four
// at most; of equal numbers the larger, which has fewer split points to do one after the other (61 layers 1.31 -> 1.19 ms).
static int key_waves(int na, int ntab) {
    int waves = 1;
    for (int w = 2; w <= kKeyWaves; ++w)
        if (key_waves_on(na, ntab, w) >= key_waves_on(na, ntab, waves)) waves = w;
    return waves;
}
// Launch shape of k_split_key for one family of one level; waves and LDS follow per launch (key_waves, key_lds).
bool plan_split_key(const Shape &sh, int Sp, int fam, SplitPlan *p) {
    int t_lo, t_hi;
    target_units(fam, Sp, sh.M, sh.n_max, &t_lo, &t_hi);
    if (fam == 0 && Sp > sh.M) return false;
    if (t_hi < t_lo) return false;
    const int cnt = t_hi - t_lo + 1;
    p->groups = cdiv(cnt, kKeyTargets);
    int most = 0, least = 0; // streaming tables of the split that has most of them, by padding and where the shorter side streams
    for (int s = 1; s < Sp; ++s) {
        int A_lo, A_hi, B_lo, B_hi;
        child_units(fam, s, sh.M, sh.n_max, &A_lo, &A_hi);
        child_units(fam, Sp - s, sh.M, sh.n_max, &B_lo, &B_hi);
        for (int g = 0; g < p->groups; ++g) {
            const int a0 = t_lo + g * kKeyTargets, a1 = imin(t_hi, a0 + kKeyTargets - 1);
            const int mA0 = imax(A_lo, a0 - B_hi), mA1 = imin(A_hi, a1 - B_lo);
            const int mB0 = imax(B_lo, a0 - A_hi), mB1 = imin(B_hi, a1 - A_lo);
            if (mA0 <= mA1 && mB0 <= mB1) {
                const int nA = mA1 - mA0 + 1, nB = mB1 - mB0 + 1;
                most = imax(most, left_streams(nA, nB, 1 << 20) ? nA : nB);
                least = imax(least, imin(nA, nB));
            }
        }
    }
    p->na = imin(cnt, kKeyTargets);
    p->full = most ? most + 8 : 1; // streaming side, one block of the stationary side
    p->range = least;              // most m of a target and split
    // The LDS of a launch is that of its split with the most streaming tables.  Where the splits of a short and a long side keep
    // one workgroup of four waves (or more) off the compute unit, their shorter side streams: as many tables as leave room for it.
    // Headline workload, time of the levels 36-43 (12 -> 16 waves) 775 -> 637 us, 55-61 (8 -> 12) 837 -> 743 us, call 6.70 ->
    // 6.53 ms.  Not for a wave more in workgroups of three (levels 62-67, 8 -> 9 waves 542 -> 653 us; 48-54, 9 -> 12 waves
    // 848 -> 918 us): the padding of the longer side costs more.  488 jobs of 12 to 160 layers, 2 to 64 nodes of 1, 2, 4 and 8 GPUs, and ten batches, against
    // sides by their padding alone: 0.94 to 1.00 of the time where it applies.
    p->cap = most;
    auto on = [&](int cap) { return key_waves_on(p->na, cap + 8, key_waves(p->na, cap + 8)); };
    if (most) {
        const int goal = on(least), had = on(most);
        if (had >= 8 && goal >= had + 4) while (on(p->cap) < goal) --p->cap;
    }
    p->ntab = most ? p->cap + 8 : 1;
    return true;
}

} // namespace oob

using namespace oob;

// The streams of an overlapped job beside the caller's.
struct Pair { hipStream_t even, odd; };

// The second stream and the events of a handle are borrowed from a pool that lives as long as the
// process and are given back when the handle is destroyed: nothing is created or destroyed per
// handle once the pool is warm (a harness that created and destroyed hundreds of handles, each
// with a stream and events of its own, ended in a host segmentation fault inside the runtime).
struct AuxPool {
    std::mutex mu;
    std::vector<hipStream_t> streams;
    std::vector<Pair> pairs;
    std::vector<hipStream_t> idle;
    std::vector<hipEvent_t> events;
};
static AuxPool &aux_pool() {
    static AuxPool *p = new AuxPool(); // never destroyed: no order-of-destruction trouble at exit
    return *p;
}
// The runtime deals streams out to its hardware queues (four by default) in turn, and work of streams on one queue does not
// overlap.  So streams are made four at a time, the third (which from the second four on gets the queue of the default stream) and
// what a pair leaves over only keep the turns in step: a pair, or three lanes, are on different queues and not on that of the default stream.
// Made as they were asked for, every second handle had both streams on one queue or one on the caller's: headline workload, six handles
// alive, 6.8, 8.8, 6.8, 9.9, 6.8, 9.9 ms a call, 6.9 ms each like this; batch of 32 jobs behind such a handle 85 and 78 ms.  (Where the
// caller makes streams in between, the turns differ, and one may still meet the caller's queue.)
static bool make_four(AuxPool &p, hipStream_t *s) {
    for (int i = 0; i < 4; ++i)
        if (hipStreamCreateWithFlags(&s[i], hipStreamNonBlocking) != hipSuccess) {
            (void)hipGetLastError();
            p.streams.insert(p.streams.end(), s, s + i);
            return false;
        }
    p.idle.push_back(s[2]);
    return true;
}
static hipStream_t borrow_stream() {
    AuxPool &p = aux_pool();
    std::lock_guard<std::mutex> lk(p.mu);
    hipStream_t s[4];
    if (p.streams.empty() && make_four(p, s)) p.streams.insert(p.streams.end(), {s[3], s[1], s[0]});
    if (p.streams.empty()) return nullptr;
    const hipStream_t one = p.streams.back();
    p.streams.pop_back();
    return one;
}
static bool borrow_pair(Pair *pair) {
    AuxPool &p = aux_pool();
    std::lock_guard<std::mutex> lk(p.mu);
    if (p.pairs.empty()) {
        hipStream_t s[4];
        if (!make_four(p, s)) return false;
        p.idle.push_back(s[3]);
        p.pairs.push_back(Pair{s[0], s[1]});
    }
    *pair = p.pairs.back();
    p.pairs.pop_back();
    return true;
}
static hipEvent_t borrow_event() {
    AuxPool &p = aux_pool();
    std::lock_guard<std::mutex> lk(p.mu);
    if (!p.events.empty()) { hipEvent_t e = p.events.back(); p.events.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
    return e;
}

// A lane is one job's worth of workspace plus the streams and events to run a job in it.  Lane 0
// serves oob_plan_templates; oob_plan_templates_batch spreads its jobs over all lanes the caller's
// workspace has room for, so that several (small) jobs fill the GPU side by side.
constexpr int kMaxLanes = 8;
struct Lane {
    hipStream_t main = nullptr;       // lanes >= 1: borrowed; lane 0 runs on the caller's stream
    bool have_aux = false;            // (false: everything on one stream)
    Pair aux;                         // streams for the inner splits of the even / odd levels, borrowed
    std::vector<hipEvent_t> ev_level; // [2 S'] "level S' selected", [2 S' + 1] "inner splits of level S' done",
                                      // borrowed
    hipEvent_t ev_join = nullptr;     // lanes >= 1: end of the lane's work in a batch, borrowed
};

struct oob_plan {
    int max_L, max_nodes, max_M;
    char *ws;
    size_t ws_bytes;
    Carve cv;
    int lanes;        // workspace_bytes / bytes of one job, at most kMaxLanes
    size_t lane_bytes;
    Lane lane[kMaxLanes];
    hipEvent_t ev_fork; // start of a batch, borrowed at the first batch
    Shape last;       // shape of the last call (for oob_plan_export_block)
    int last_lane;    // and the lane it ran in
    bool have_last;
    hipEvent_t ev_begin, ev_end; // optional: recorded around the level launches
    bool timed;
    int opt_plain, opt_xcd, opt_one_stream, opt_select8_from, opt_fuse_from, opt_overlap_from, opt_small_state; // oob_plan_set_option
};

#define OOB_HIP_CHECK(expr)                                                                   \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess) {                                                               \
            fprintf(stderr, "oob_plan: %s failed: %s\n", #expr, hipGetErrorString(e_));       \
            return OOB_EHIP;                                                                  \
        }                                                                                     \
    } while (0)

extern "C" int oob_plan_max_stages(int L, int n_max, int gpus_per_node, int microbatches) {
    if (L < 1 || n_max < 1 || gpus_per_node < 1 || microbatches < 0) return OOB_EINVAL;
    return smax_of(L, n_max, gpus_per_node, microbatches);
}

static bool dims_ok(int L, int nodes, int M) {
    return L >= 1 && L <= OOB_MAX_L && nodes >= 1 && nodes <= OOB_MAX_NODES && M >= 1 && M <= OOB_MAX_GPUS;
}

extern "C" size_t oob_plan_workspace_size(int max_L, int max_nodes, int max_gpus_per_node) {
    if (!dims_ok(max_L, max_nodes, max_gpus_per_node)) return 0;
    return carve(max_L, max_nodes, max_gpus_per_node).total;
}

extern "C" int oob_plan_create(oob_plan **h, int max_L, int max_nodes, int max_gpus_per_node,
                               void *dev_workspace, size_t workspace_bytes) {
    if (!h) return OOB_EINVAL;
    *h = nullptr;
    if (!dims_ok(max_L, max_nodes, max_gpus_per_node) || !dev_workspace) return OOB_EINVAL;
    if (((uintptr_t)dev_workspace & 255) != 0) return OOB_EINVAL;
    const Carve cv = carve(max_L, max_nodes, max_gpus_per_node);
    if (workspace_bytes < cv.total) return OOB_ECAPACITY;
    oob_plan *p = new (std::nothrow) oob_plan();
    if (!p) return OOB_EINVAL;
    p->max_L = max_L; p->max_nodes = max_nodes; p->max_M = max_gpus_per_node;
    p->ws = (char *)dev_workspace; p->ws_bytes = workspace_bytes; p->cv = cv; p->have_last = false;
    p->ev_begin = nullptr; p->ev_end = nullptr; p->timed = false;
    p->lane_bytes = align_up(cv.total);
    p->lanes = (int)std::min<size_t>(kMaxLanes, std::max<size_t>(1, workspace_bytes / p->lane_bytes));
    p->ev_fork = nullptr; p->last_lane = 0;
    p->opt_plain = p->opt_xcd = p->opt_one_stream = 0;
    p->opt_select8_from = kSelect8From; p->opt_fuse_from = kFuseFrom; p->opt_overlap_from = kOverlapFrom; p->opt_small_state = kSmallState;
    *h = p;
    return OOB_OK;
}

extern "C" int oob_plan_destroy(oob_plan *h) {
    if (!h) return OOB_EINVAL;
    if (h->ev_begin) { (void)hipEventDestroy(h->ev_begin); (void)hipEventDestroy(h->ev_end); }
    { // the caller has waited for the handle's work: its stream and events go back to the pool
        AuxPool &p = aux_pool();
        std::lock_guard<std::mutex> lk(p.mu);
        for (Lane &ln : h->lane) {
            for (hipEvent_t e : ln.ev_level) p.events.push_back(e);
            if (ln.ev_join) p.events.push_back(ln.ev_join);
            if (ln.have_aux) p.pairs.push_back(ln.aux);
            if (ln.main) p.streams.push_back(ln.main);
        }
        if (h->ev_fork) p.events.push_back(h->ev_fork);
    }
    delete h;
    return OOB_OK;
}

static Tables make_tables(const oob_plan *h, int lane, const Shape &sh, int *status) {
    Tables t;
    char *ws = h->ws + (size_t)lane * h->lane_bytes;
    t.sh = sh;
    t.NB = nblocks_of(sh.L);
    t.coff = col_shift(sh.L);
    t.tab_recs = tri_blocks(t.NB) * 64;
    t.inv_M = inverse_of(sh.M);
    t.rec = (Rec *)(ws + h->cv.rec);
    t.partT = (double *)(ws + h->cv.partT);
    t.key = (unsigned long long *)(ws + h->cv.partT);
    t.partK = (int *)(ws + h->cv.partK);
    t.flags = (int *)(ws + h->cv.flags);
    t.seg_tab = (int2 *)(ws + h->cv.seg_tab);
    t.seg_stride = seg_count_bound(sh.L);
    t.status = status;
    return t;
}

static bool out_ok(const oob_templates *o) {
    return o && o->feasible && o->S && o->kstar && o->T && o->T1 && o->T2 && o->T3 && o->tmax &&
           o->stage_off && o->stage_begin && o->stage_gpus && o->cover_hdr && o->cover_maxpipes &&
           o->status;
}

// The splits s0, s0 + sstep, ... (scount of them) of level S.
struct SplitRange { int s0, sstep, scount; };

// A keyed launch: the target groups of family `fam` (gz of them) and, in a launch for both families
// of a low level, those of the whole-node family behind them (`groups` in all); at most ntab tables
// staged per split point, na targets per group.
struct KeyLaunch { int fam, gz, groups, ntab, na, cap; };
// Most tables per split point the keyed kernel serves: with a full group of targets four waves then still fit a
// compute unit, in a workgroup of 140 KB.  Measured against the plain kernel, most tables, layers x nodes x GPUs per node:
// 76, 150 x 150 x 8: 109 and 329 ms; 82, 140 x 140 x 64: 137 and 452 ms; 99, 176 x 176 x 8: 313 and 833 ms; 120, 200 x 200 x 8:
// 747 and 1 790 ms; 136, 240 x 200 x 8: 2.67 and 5.50 s.
constexpr int kKeyTables = 144;
static size_t key_lds(int na, int ntab) { return (size_t)na * 512 + (size_t)key_waves(na, ntab) * ntab * 192; }
static void launch_split_key(const Tables &t, int S, const KeyLaunch &kl, int NT, int xcd, SplitRange sr, hipStream_t st) {
    KeyArgs ka;
    ka.na = kl.na; ka.cap = kl.cap;
    ka.Sp = S; ka.fam0 = kl.fam; ka.gz = kl.gz; ka.NT = NT; ka.s0 = sr.s0; ka.sstep = sr.sstep;
    ka.t_lo1 = imax(2, cdiv(S, t.sh.M)); ka.dlo = dlo_of(S, t.sh.M); ka.pack = kKeyPack; ka.xcd = xcd;
    hipLaunchKernelGGL(k_split_key, dim3(seg_count(t.sh.L, S), sr.scount, kl.groups), dim3(key_waves(kl.na, kl.ntab) * 64), key_lds(kl.na, kl.ntab), st, t, ka);
}
// The keyed launches of the splits `sr` of a level: one per family, or one for both.
static void launch_split_keys(const Tables &t, int S, const bool *have, const SplitPlan *kp, int NT, int xcd,
                              SplitRange sr, hipStream_t st) {
    if (sr.scount < 1) return;
    KeyLaunch kl[2];
    for (int fam = 0; fam < 2; ++fam)
        if (have[fam])
            kl[fam] = KeyLaunch{fam, kp[fam].groups, kp[fam].groups, kp[fam].ntab, kp[fam].na, kp[fam].cap};
    if (have[0] && have[1]) {
        const KeyLaunch both{0, kl[0].groups, kl[0].groups + kl[1].groups, imax(kl[0].ntab, kl[1].ntab),
                             imax(kl[0].na, kl[1].na), imax(kl[0].cap, kl[1].cap)};
        launch_split_key(t, S, both, NT, xcd, sr, st);
        return;
    }
    for (int fam = 0; fam < 2; ++fam)
        if (have[fam]) launch_split_key(t, S, kl[fam], NT, xcd, sr, st);
}

template <int PC>
static void launch_split(const Tables &t, int S, int fam, const SplitPlan &sp, int NT, int NAall,
                         hipStream_t st) {
    if (sp.lds > kLdsPrefer) // beyond the default dynamic-LDS limit of a launch
        (void)hipFuncSetAttribute((const void *)k_split<PC>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)kLdsLimit);
    hipLaunchKernelGGL(k_split<PC>, dim3(NT, S - 1, sp.groups), dim3(sp.waves * 64), sp.lds, st, t, S, fam,
                       NT, NAall);
}

// One job in lane `ln` of the handle, enqueued on `st` (and on the lane's second stream when the
// levels overlap).
static int enqueue_job(oob_plan *h, int ln, bool want_overlap, const oob_profile *profile, int L, int n_min,
                       int n_max, int gpus_per_node, int microbatches, int64_t mem_cap, int f,
                       oob_templates *out, hipStream_t st) {
    if (!h || !profile || !out_ok(out)) return OOB_EINVAL;
    Lane &lane = h->lane[ln];
    if (!profile->fwd_ns || !profile->bwd_ns || !profile->mem_bytes || !profile->boundary_ns) return OOB_EINVAL;
    if (L < 1 || n_min < 1 || n_min > n_max || gpus_per_node < 1 || microbatches < 0 || f < 0 || mem_cap <= 0)
        return OOB_EINVAL;
    if (L > h->max_L || n_max > h->max_nodes || gpus_per_node > h->max_M) return OOB_ECAPACITY;
    if ((long long)n_max * ((long long)f + 1) > (1 << 24)) return OOB_ECAPACITY;
    const int M = gpus_per_node;
    if (table_count(L, M, n_max, microbatches) * tri_blocks(nblocks_of(L)) * 64 > h->cv.recs ||
        part_slots(L, M, n_max, microbatches) > h->cv.slots)
        return OOB_ECAPACITY;
    Shape sh;
    sh.L = L; sh.M = M; sh.n_min = n_min; sh.n_max = n_max; sh.Nb = microbatches; sh.f = f;
    sh.cap = mem_cap; sh.count = n_max - n_min + 1;
    sh.Smax = smax_of(L, n_max, M, microbatches);
    // launch shapes first, so that nothing is enqueued when a level cannot be staged in LDS
    // a level stages more tables than the keyed kernel serves (or the debug knob says so): plain kernel everywhere
    int force_plain = h->opt_plain != 0;
    size_t lds = 0; // of the largest keyed launch
    for (int S = 2; S <= sh.Smax; ++S) {
        int ntab = 0, na = 0, full = 0;
        for (int fam = 0; fam < 2; ++fam) {
            SplitPlan sp;
            if (plan_split_key(sh, S, fam, &sp)) { ntab = imax(ntab, sp.ntab); na = imax(na, sp.na); full = imax(full, sp.full); }
        }
        if (full > kKeyTables) force_plain = 1;
        else if (ntab) lds = std::max(lds, key_lds(na, ntab));
    }
    if (!force_plain && lds > kLdsPrefer) // beyond the default dynamic-LDS limit of a launch
        OOB_HIP_CHECK(hipFuncSetAttribute((const void *)k_split_key, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit));
    if (force_plain)
        for (int S = 2; S <= sh.Smax; ++S)
            for (int fam = 0; fam < 2; ++fam) {
                SplitPlan sp;
                if (plan_split(sh, S, fam, &sp) && sp.lds > kLdsLimit) return OOB_ECAPACITY;
            }
    const Tables t = make_tables(h, ln, sh, (int *)out->status);
    // states and candidates; the levels worth an overlap (below)
    int ov_lo = sh.Smax + 1, ov_hi = 0;
    signed char small[OOB_MAX_L + 1]; // levels done by one launch: the columns of its workgroups (lgC), else -1
    out->states = out->candidates = 0;
    for (int S = 1; S <= sh.Smax; ++S) {
        long long states, cands;
        int most;
        level_counts(sh, S, &states, &cands, &most);
        out->states += states; out->candidates += cands;
        if (S >= 4 && cands >= h->opt_overlap_from * 1000ll) { ov_lo = imin(ov_lo, S); ov_hi = S; }
        const long long widest = (long long)most * (L - S + 1);
        small[S] = S >= 2 && most <= kSmallPairs && widest <= h->opt_small_state && cands <= kSmallLevel ? small_columns(sh, S, widest) : -1;
    }
    if (table_count(L, M, n_max, microbatches) * tri_blocks(nblocks_of(L)) * 64 * (long long)sizeof(Rec) >= 1ll << 32 || force_plain)
        std::fill(small, small + sh.Smax + 1, (signed char)-1); // its offsets are 32 bits

    const long long slot_stride = h->cv.slots * 64; // distance between the two buffers of per-split minima
    long long keys = 0; // of the level that has most of them
    for (int S = 2; S <= sh.Smax; ++S) keys = std::max(keys, (long long)(dhi_of(S, M, n_max) - dlo_of(S, M) + 1) * tile_count(L, S) * 64);
    bool overlap = want_overlap && !force_plain && ov_lo <= ov_hi;
    int how = force_plain;
    for (int S = 2; S <= sh.Smax; ++S) how += small[S] >= 0 ? 1 << 1 : overlap && S >= ov_lo && S <= ov_hi ? 1 << (1 + kHowBits) : 0;
    const int ones = M * ((tile_count(L, 1) + 3) / 4);
    hipLaunchKernelGGL(k_prepare, dim3((unsigned)(1 + ones + imax(sh.Smax - 1, 0) + (2 * keys + kSetupThreads - 1) / kSetupThreads)),
                       dim3(kSetupThreads), 0, st, t, *profile, how, h->opt_xcd, ones, slot_stride, keys);
    // Levels.  Level S' depends on the lower levels like this: its inner splits 2 <= s <= S'-2 read the
    // levels up to S'-2 only, its two outer splits (s = 1 and S'-1) read level S'-1, and its select
    // needs all its splits.  So the chain that cannot be shortened is outer splits -> select ->
    // outer splits of the next level ..., two small launches per level, and it runs on the caller's
    // stream.  The inner splits, nearly all of the arithmetic, run on two streams of the library (even
    // and odd levels), each launch waiting for the select of level S'-2 and awaited by the select of its
    // own level; they fill the machine around the chain.  Each parity has its own buffer of
    // keys (a select hands its buffer back reset before the inner splits of level S'+2 start).
    // That pays from the first to the last level of at least opt_overlap_from thousand candidates.  The other levels
    // put all their splits into one launch on the caller's stream: a level takes 10-25 us there, and the two event
    // records, the two waits and the third launch of an overlapped one occupy the host for longer (one stream
    // throughout, against three: 26 layers 312 and 732 us, 61 layers 1.62 and 1.78 ms, headline workload 10.5 and
    // 7.5 ms; the line at 0, 20, 40, 80 million candidates: headline workload 7.47, 7.60, 7.69, 7.89 ms).
    if (overlap && !lane.have_aux) lane.have_aux = borrow_pair(&lane.aux);
    if (overlap && lane.have_aux) {
        while ((int)lane.ev_level.size() < 2 * sh.Smax + 2) {
            hipEvent_t e = borrow_event();
            if (!e) break;
            lane.ev_level.push_back(e);
        }
    }
    overlap = overlap && lane.have_aux && (int)lane.ev_level.size() >= 2 * sh.Smax + 2;
    const bool timed = ln == 0 && h->ev_begin;
    if (timed) OOB_HIP_CHECK(hipEventRecord(h->ev_begin, st));
    for (int S = 2; S <= sh.Smax; ++S) {
        const int NAall = dhi_of(S, M, n_max) - dlo_of(S, M) + 1;
        if (NAall <= 0) continue;
        const int NT = tile_count(L, S);
        if (small[S] >= 0) {
            hipLaunchKernelGGL(k_level_small, dim3(NT, NAall, 8 << (3 - small[S])), dim3(kSmallThreads), 0, st, t, S, (int)small[S]);
            if (overlap && S + 2 >= ov_lo && S + 2 <= ov_hi) OOB_HIP_CHECK(hipEventRecord(lane.ev_level[2 * S], st));
            continue;
        }
        Tables tl = t; // this level's buffer of per-split minima
        tl.partT = t.partT + (S & 1) * slot_stride;
        tl.key = t.key + (S & 1) * slot_stride;
        SplitPlan sp[2], kp[2];
        bool have[2];
        for (int fam = 0; fam < 2; ++fam) {
            have[fam] = plan_split(sh, S, fam, &sp[fam]) && plan_split_key(sh, S, fam, &kp[fam]);
        }
        const bool inner = overlap && S >= ov_lo && S <= ov_hi;
        const bool many = want_overlap && !inner && have[1] && kp[1].range > kSel8Range && NT * NAall * 8 <= kSel8Waves;
        if (inner) {
            hipStream_t sx = (S & 1) ? lane.aux.odd : lane.aux.even;
            OOB_HIP_CHECK(hipStreamWaitEvent(sx, lane.ev_level[2 * (S - 2)], 0)); // select of level S'-2
            launch_split_keys(tl, S, have, kp, NT, h->opt_xcd, SplitRange{2, 1, S - 3}, sx);
            OOB_HIP_CHECK(hipEventRecord(lane.ev_level[2 * S + 1], sx));
        }
        // the outer splits: launches of their own, or evaluated by the select kernel itself
        const bool fuse = !force_plain && S >= h->opt_fuse_from;
        if (!force_plain) {
            SplitRange sr = inner ? SplitRange{1, S - 2, 2} : SplitRange{1, 1, S - 1};
            if (fuse) sr = inner ? SplitRange{1, 1, 0} : SplitRange{2, 1, S - 3};
            launch_split_keys(tl, S, have, kp, NT, h->opt_xcd, sr, st);
        }
        for (int fam = 0; fam < 2 && force_plain; ++fam) {
            if (!have[fam]) continue;
            if (sp[fam].pc == 4) launch_split<4>(tl, S, fam, sp[fam], NT, NAall, st);
            else if (sp[fam].pc == 2) launch_split<2>(tl, S, fam, sp[fam], NT, NAall, st);
            else launch_split<1>(tl, S, fam, sp[fam], NT, NAall, st);
        }
        if (inner) OOB_HIP_CHECK(hipStreamWaitEvent(st, lane.ev_level[2 * S + 1], 0));
        if (force_plain) hipLaunchKernelGGL(k_select, dim3(NT, NAall), dim3(64), 0, st, tl, S, NT, NAall);
        else if (fuse) hipLaunchKernelGGL((k_select_key<8, true>), dim3(NT, NAall, 8), dim3(64), 0, st, tl, S, NT, NAall);
        else if (S >= h->opt_select8_from || many) hipLaunchKernelGGL((k_select_key<8, false>), dim3(NT, NAall, 8), dim3(64), 0, st, tl, S, NT, NAall);
        else hipLaunchKernelGGL((k_select_key<kSelLanes, false>), dim3(NT, NAall, kSelLanes), dim3(64), 0, st, tl, S, NT, NAall);
        if (overlap && S + 2 >= ov_lo && S + 2 <= ov_hi) OOB_HIP_CHECK(hipEventRecord(lane.ev_level[2 * S], st));
    }
    if (timed) { OOB_HIP_CHECK(hipEventRecord(h->ev_end, st)); h->timed = true; }
    hipLaunchKernelGGL(k_pick, dim3(sh.count), dim3(64), 0, st, t, *out);
    hipLaunchKernelGGL(k_backtrack, dim3(sh.count + 1), dim3(128), 0, st, t, *out, sh.count > f + 1 ? sh.count : f + 1);
    OOB_HIP_CHECK(hipGetLastError());
    h->last = sh;
    h->last_lane = ln;
    h->have_last = true;
    return OOB_OK;
}

extern "C" int oob_plan_templates(oob_plan *h, const oob_profile *profile, int L, int n_min, int n_max,
                                  int gpus_per_node, int microbatches, int64_t mem_cap, int f,
                                  oob_templates *out, void *stream) {
    return enqueue_job(h, 0, h && !h->opt_one_stream, profile, L, n_min, n_max, gpus_per_node, microbatches, mem_cap, f,
                       out, (hipStream_t)stream);
}

extern "C" int oob_plan_templates_batch(oob_plan *h, int count, const oob_profile *profiles, const int *L,
                                        const int *n_min, const int *n_max, const int *gpus_per_node,
                                        const int *microbatches, const int64_t *mem_cap, const int *f,
                                        oob_templates *outs, void *stream) {
    if (!h || count < 0 || (count > 0 && (!profiles || !L || !n_min || !n_max || !gpus_per_node ||
                                           !microbatches || !mem_cap || !f || !outs)))
        return OOB_EINVAL;
    const int want_overlap = !h->opt_one_stream, lane_overlap = kBatchOverlap, max_lanes = kBatchLanes;
    hipStream_t st = (hipStream_t)stream;
    // Lanes: job i runs in lane i mod K, the jobs of a lane one after the other on the lane's own
    // stream, the lanes side by side.  Lane 0 is the caller's stream; the others start after what
    // the caller has enqueued so far (fork event) and the caller's stream waits for them at the end.
    int K = std::max(1, std::min(std::min(h->lanes, max_lanes), count));
    if (K > 1 && !h->ev_fork) h->ev_fork = borrow_event();
    if (K > 1 && !h->ev_fork) K = 1;
    for (int ln = 1; ln < K; ++ln) {
        Lane &lane = h->lane[ln];
        if (!lane.main) lane.main = borrow_stream();
        if (!lane.ev_join) lane.ev_join = borrow_event();
        if (!lane.main || !lane.ev_join) { K = ln; break; }
    }
    if (K > 1) {
        OOB_HIP_CHECK(hipEventRecord(h->ev_fork, st));
        for (int ln = 1; ln < K; ++ln) OOB_HIP_CHECK(hipStreamWaitEvent(h->lane[ln].main, h->ev_fork, 0));
    }
    int rc = OOB_OK;
    for (int i = 0; i < count && rc == OOB_OK; ++i) {
        const int ln = i % K;
        rc = enqueue_job(h, ln, K > 1 ? lane_overlap != 0 : want_overlap != 0, &profiles[i], L[i], n_min[i], n_max[i],
                         gpus_per_node[i], microbatches[i], mem_cap[i], f[i], &outs[i], ln ? h->lane[ln].main : st);
    }
    for (int ln = 1; ln < K; ++ln) { // also after an error: the caller's stream covers all that was enqueued
        OOB_HIP_CHECK(hipEventRecord(h->lane[ln].ev_join, h->lane[ln].main));
        OOB_HIP_CHECK(hipStreamWaitEvent(st, h->lane[ln].ev_join, 0));
    }
    return rc;
}

extern "C" int oob_plan_set_option(oob_plan *h, int option, int value) {
    if (!h) return OOB_EINVAL;
    switch (option) {
    case OOB_OPT_PLAIN_SPLIT: h->opt_plain = value != 0; break;
    case OOB_OPT_XCD_ORDER: h->opt_xcd = value != 0; break;
    case OOB_OPT_ONE_STREAM: h->opt_one_stream = value != 0; break;
    case OOB_OPT_SELECT8_FROM: h->opt_select8_from = value; break;
    case OOB_OPT_FUSE_FROM: h->opt_fuse_from = value; break;
    case OOB_OPT_OVERLAP_FROM: h->opt_overlap_from = value; break;
    case OOB_OPT_SMALL_STATE: h->opt_small_state = value; break;
    default: return OOB_EINVAL;
    }
    return OOB_OK;
}

extern "C" int oob_plan_level_timing(oob_plan *h, int enable) {
    if (!h) return OOB_EINVAL;
    if (enable && !h->ev_begin) {
        OOB_HIP_CHECK(hipEventCreate(&h->ev_begin));
        OOB_HIP_CHECK(hipEventCreate(&h->ev_end));
    } else if (!enable && h->ev_begin) {
        (void)hipEventDestroy(h->ev_begin); (void)hipEventDestroy(h->ev_end);
        h->ev_begin = h->ev_end = nullptr;
    }
    h->timed = false;
    return OOB_OK;
}

extern "C" int oob_plan_last_level_ms(oob_plan *h, float *ms) {
    if (!h || !ms || !h->ev_begin || !h->timed) return OOB_EINVAL;
    OOB_HIP_CHECK(hipEventSynchronize(h->ev_end));
    OOB_HIP_CHECK(hipEventElapsedTime(ms, h->ev_begin, h->ev_end));
    return OOB_OK;
}

// Measurement: sixteen independent chains of 32-bit add / compare / select per lane, the
// operation mix the roofline of the level kernels is quoted in.  3 lane-operations per chain step.
__global__ void __launch_bounds__(256) k_valu_peak(int *sink, int iters, int a, int b) {
    int v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = threadIdx.x + i * a;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int w = v[i] + a;
            v[i] = w > b ? w : v[i];
        }
    }
    int r = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) r ^= v[i];
    if (r == 0x7fffffff) sink[0] = r; // keeps the chains alive; practically never taken
}

// Measurement: the step of k_split_key without LDS, keys and addresses: eight candidates by four_candidates, four
// vector instructions each (compare, add, the other add under its mask, min), plus the three adds that change the
// step's streaming values.  kPeakStep lane-instructions per step.
constexpr double kPeakStep = 8 * 4 + 3;
__global__ void __launch_bounds__(256) k_valu_peak_f64(double *sink, int iters, double a, double b) {
    double bb2[8], bbt[8], btm[8], acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        bb2[i] = a * (threadIdx.x + i); bbt[i] = b * (threadIdx.x + 2 * i); btm[i] = a * b * (3 * i + (threadIdx.x & 7));
        acc[i] = 1e300;
    }
    double2 p = make_double2(a, b);
    double atm = a + b;
    for (int it = 0; it < iters; ++it) {
        four_candidates<false>(acc[0], acc[1], acc[2], acc[3], bb2, bbt, btm, p, atm);
        four_candidates<false>(acc[4], acc[5], acc[6], acc[7], bb2 + 4, bbt + 4, btm + 4, p, atm);
        p.x += a; p.y += b; atm += a;
    }
    double r = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) r += acc[i];
    if (r == 12345.678) sink[0] = r; // keeps the chains alive; practically never taken
}

// Host-side check of the table layout and the task lists for L layers (no GPU involved): every state
// (S', u, v) lies in exactly one enumerated block of its level and at a record of its own, every
// enumerated block holds a state, the segments of a block partition its split range into parts of at
// least one split point, and the counts stay within the bounds that size a workspace.
extern "C" int oob_plan_layout_selftest(int L) {
    if (L < 1 || L > OOB_MAX_L) return OOB_EINVAL;
    const int NB = nblocks_of(L), c = col_shift(L), recs = tri_blocks(NB) * 64;
    if ((L + c + 1) % 8 != 0 || (L + c) / 8 != NB - 1) return 1;
    static_assert(OOB_MAX_L <= kOverMBelow && OOB_MAX_GPUS <= 64, "over_M divides numbers of levels by GPUs per node");
    for (int M = 1; M <= OOB_MAX_GPUS; ++M)
        for (int k = 0; k < kOverMBelow; ++k)
            if (over_M(k, inverse_of(M)) != k / M) return 13;
    for (int M = 1; M <= OOB_MAX_GPUS; ++M) // the closed form of the levels' tables
        for (int n_max = 1; n_max <= imin(L, OOB_MAX_NODES); n_max += 1 + n_max / 3) {
            int tab = 0;
            for (int S = 1; S <= imin(L, n_max * M); ++S) {
                const Level lv = level_of(S, M, n_max, inverse_of(M));
                const int nd = dhi_of(S, M, n_max) - dlo_of(S, M) + 1;
                if (lv.base + dlo_of(S, M) != tab || lv.least != cdiv(S, M) || nd < 1) return 12;
                tab += nd;
            }
        }
    std::vector<int> owner((size_t)(L + 1) * (L + 1));
    std::vector<char> used(recs);
    for (int u = 0; u <= L; ++u) // records of distinct (u, v) are distinct and inside the table
        for (int v = u; v <= L; ++v) {
            const int o = rec_off(u, v, c, NB);
            if (o < 0 || o >= recs || used[o]) return 2;
            used[o] = 1;
        }
    for (int S = 1; S <= L; ++S) {
        std::fill(owner.begin(), owner.end(), -1);
        const int nt = tile_count(L, S);
        if (nt > tile_count_bound(L, S)) return 3;
        int segs = 0;
        for (int t = 0; t < nt; ++t) {
            int ub, vb;
            tile_decode(L, S, t, &ub, &vb);
            if (ub < 0 || vb < ub || vb >= NB) return 4;
            const int kr = tile_krange(L, S, ub, vb);
            if (kr < 1 || tile_vmax(L, vb) > L) return 5;
            const int n = seg_n(kr, seg_target(L, S));
            int next = 0;
            for (int j = 0; j < n; ++j) {
                int ofs, len;
                seg_span(kr, n, j, &ofs, &len);
                if (ofs != next || len < 1) return 6;
                next = ofs + len;
            }
            if (next != kr) return 6;
            segs += n;
            int states = 0;
            for (int u = ub * 8; u < ub * 8 + 8; ++u)
                for (int v = vb * 8 - c; v <= vb * 8 + 7 - c; ++v) {
                    if (u >= L || v < 0 || v > L || v - u < S) continue;
                    if (owner[(size_t)u * (L + 1) + v] != -1) return 7;
                    owner[(size_t)u * (L + 1) + v] = t;
                    if (rec_off(u, v, c, NB) != tri_index(ub, vb, NB) * 64 + ((u - ub * 8) << 3) + (v + c - vb * 8)) return 8;
                    ++states;
                }
            if (states == 0) return 9;
        }
        for (int u = 0; u < L; ++u)
            for (int v = u + S; v <= L; ++v)
                if (owner[(size_t)u * (L + 1) + v] < 0) return 10;
        if (S >= 2 && (segs != seg_count(L, S) || segs > seg_count_bound(L))) return 11;
    }
    return 0;
}

// Copies flags[0..3] of the last call to a device array (tests: which split kernel ran).
__global__ void k_export_flags(const int *flags, int *dst) {
    if (threadIdx.x < 4) dst[threadIdx.x] = flags[threadIdx.x];
}

extern "C" int oob_plan_export_flags(oob_plan *h, int32_t *flags, void *stream) {
    if (!h || !h->have_last || !flags) return OOB_EINVAL;
    hipLaunchKernelGGL(k_export_flags, dim3(1), dim3(64), 0, (hipStream_t)stream, (const int *)(h->ws + (size_t)h->last_lane * h->lane_bytes + h->cv.flags),
                       (int *)flags);
    OOB_HIP_CHECK(hipGetLastError());
    return OOB_OK;
}

extern "C" int oob_plan_export_block(oob_plan *h, int S, int delta, double *T, double *T1, double *tmax,
                                     double *T3, int32_t *kstar, int32_t *choice, void *stream) {
    if (!h || !h->have_last || !T || !T1 || !tmax || !T3 || !kstar || !choice) return OOB_EINVAL;
    const Shape &sh = h->last;
    if (S < 1 || S > sh.Smax) return OOB_EINVAL;
    if (delta < dlo_of(S, sh.M) || delta > dhi_of(S, sh.M, sh.n_max)) return OOB_EINVAL;
    const Tables t = make_tables(h, h->last_lane, sh, nullptr);
    const int n = sh.L - S + 1;
    hipLaunchKernelGGL(k_export, dim3((n * n + 255) / 256), dim3(256), 0, (hipStream_t)stream, t, S, delta, T,
                       T1, tmax, T3, (int *)kstar, (int *)choice);
    OOB_HIP_CHECK(hipGetLastError());
    return OOB_OK;
}

// Measured vector-ALU peak of this GPU in lane-operations per second, for comparison with the nominal
// 256 CUs x 64 lanes x clock: 32-bit add / compare / select (f64_mix = 0) or the fp64 instructions of a
// candidate of the keyed split kernel (f64_mix = 1).
static int valu_peak(oob_plan *h, void *stream, double *lane_ops_per_s, int f64_mix) {
    if (!h || !lane_ops_per_s) return OOB_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0, e1;
    OOB_HIP_CHECK(hipEventCreate(&e0));
    OOB_HIP_CHECK(hipEventCreate(&e1));
    const int iters = f64_mix ? 6000 : 20000, grid = 256 * 32; // 32 workgroups of 4 waves per compute unit
    int *sink = (int *)(h->ws + h->cv.flags) + 32; // spare words of the flags array (8-byte aligned)
    for (int pass = 0; pass < 2; ++pass) { // warm-up, then the timed launch
        if (pass) OOB_HIP_CHECK(hipEventRecord(e0, st));
        if (f64_mix) hipLaunchKernelGGL(k_valu_peak_f64, dim3(grid), dim3(256), 0, st, (double *)sink, pass ? iters : 100, 1.0, 3.0);
        else         hipLaunchKernelGGL(k_valu_peak, dim3(grid), dim3(256), 0, st, sink, pass ? iters : 100, 1, 1 << 30);
    }
    OOB_HIP_CHECK(hipEventRecord(e1, st));
    OOB_HIP_CHECK(hipEventSynchronize(e1));
    float ms = 0.f;
    OOB_HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *lane_ops_per_s = (double)grid * 256 * (f64_mix ? kPeakStep : 16.0 * 3) * iters / (ms * 1e-3);
    return OOB_OK;
}
extern "C" int oob_plan_valu_peak(oob_plan *h, void *stream, double *lane_ops_per_s) {
    return valu_peak(h, stream, lane_ops_per_s, 0);
}
extern "C" int oob_plan_valu_peak_f64(oob_plan *h, void *stream, double *lane_ops_per_s) {
    return valu_peak(h, stream, lane_ops_per_s, 1);
}
