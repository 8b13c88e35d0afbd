// Pipeline-instantiation enumeration (Section 4.2.1, Eq. 5 of the Oobleck paper) for gfx950.
//
// Eq. 5 builds lists by concatenation; on the GPU the lists are never built.  Replacing every
// list by its length turns the equation into a counting recurrence, and the position of a
// vector inside X(p, N') then determines the vector: at (p', N') a position below
// |X(p'-1, N')| lies in the copied part (x_{p'-1} is final), any other position lies in the
// theta part (one more pipeline of size n_{p'-1}, continue at N' - n_{p'-1}).  The paper's
// second requirement (at least f+1 pipelines) filters the final list without reordering it;
// carrying "q more pipelines are still required" as a third index of the count table makes the
// filtered lists directly addressable:
//     C(p', N', q) = C(p'-1, N', q) + C(p', N' - n_{p'-1}, max(q-1, 0)),   C(0, 0, 0) = 1.
// Every output vector is then produced by one lane, independently of all others, and stored
// structure-of-arrays so that a wave writes 128 contiguous bytes per template.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <atomic>
#include <mutex>
#include <type_traits>

#include "oob_inst.h"
#include "oob_plan.h"

namespace oob_inst {

constexpr long long kSat = 1ll << 62; // counts saturate here; a saturated total is an error
constexpr int kGroup = 8;             // counts a lane reads at once

// Count table: row (N', q) holds C(j, N', q) for j = 0..p, padded to whole groups, so that the
// counts a position is compared with (same N', same q, descending j) are contiguous.
struct Spec {
    const int *sizes; // may be null: consecutive from n0
    int p, n0, N_lo, N_hi, Q, R; // Q = f + 1; R = row length
    long long *cnt;              // [(N_hi+1)][(Q+1)][R]
    unsigned *cnt32;             // the same table in 32 bits, valid if *narrow
    int *narrow;                 // [1] every count is below 2^32
};
constexpr size_t kHeaderBytes = 256; // the workspace starts with `narrow`, the two tables follow

__host__ __device__ inline int row_len(int p) { return (p + 1 + kGroup - 1) / kGroup * kGroup; }
__device__ __forceinline__ int size_of(const Spec &s, int j) { return s.sizes ? s.sizes[j] : s.n0 + j; }
__device__ __forceinline__ long long sat_add(long long a, long long b) {
    const unsigned long long c = (unsigned long long)a + (unsigned long long)b; // both <= 2^62: fits 64 bits
    return c > (unsigned long long)kSat ? kSat : (long long)c;
}

// One workgroup.  Plane j of the table (all N', q) needs plane j-1 only, and inside a plane the
// recurrence along N' unrolls into a sum over the number i of size-n pipelines:
//     C(j, N', q) = sum_{i >= 0, i n <= N'} C(j-1, N' - i n, max(q - i, 0)),
// so all entries of a plane are independent: one barrier per template size.  With IN_LDS the
// previous and the current plane live in LDS (two planes of (N_hi+1)(Q+1) counts); otherwise
// the previous plane is read back from the table.  Used where k_inst_count_ring does not fit.
template <bool IN_LDS>
__global__ void __launch_bounds__(1024) k_inst_count(Spec s, long long *offsets, int *status, int keep_wide) {
    HIP_DYNAMIC_SHARED(long long, s_dyn) // IN_LDS: two planes; then reused for the prefix sum
    __shared__ int s_bad;
    __shared__ unsigned long long s_max;
    const int QQ = s.Q + 1, plane = (s.N_hi + 1) * QQ, len = s.N_hi - s.N_lo + 1;
    if (threadIdx.x == 0) { s_bad = 0; s_max = 0; }
    __syncthreads();
    for (int j = threadIdx.x; j < s.p; j += blockDim.x) {
        const int n = size_of(s, j);
        if (n < 1 || (j > 0 && n <= size_of(s, j - 1))) s_bad = 1;
    }
    for (int e = threadIdx.x; e < plane; e += blockDim.x) { // C(0, ., .)
        const long long c = e == 0 ? 1 : 0;
        s.cnt[(long long)e * s.R] = c;
        if (IN_LDS) s_dyn[e] = c;
        // the padding of a row compares greater than any list position
        for (int j = s.p + 1; j < s.R; ++j) s.cnt[(long long)e * s.R + j] = 0x7FFFFFFFFFFFFFFFll;
    }
    __syncthreads();
    if (s_bad) { // uniform: every thread leaves here
        for (int i = threadIdx.x; i <= len; i += blockDim.x) offsets[i] = 0;
        if (threadIdx.x == 0) { *status = OOB_EINVAL; *s.narrow = 0; }
        return;
    }
    long long mine = 1; // largest count this thread has written
    for (int j = 1; j <= s.p; ++j) {
        const int n = size_of(s, j - 1);
        const long long *prev = IN_LDS ? s_dyn + ((j - 1) & 1) * plane : s.cnt + (j - 1);
        const long long pstride = IN_LDS ? 1 : s.R;
        long long *cur = s_dyn + (j & 1) * plane;
        for (int e = threadIdx.x; e < plane; e += blockDim.x) {
            const int N = e / QQ, q = e - N * QQ;
            long long sum = 0;
            for (int i = 0, Ni = N; Ni >= 0; ++i, Ni -= n) {
                const int qi = q - i > 0 ? q - i : 0;
                sum = sat_add(sum, prev[(long long)(Ni * QQ + qi) * pstride]);
            }
            s.cnt[(long long)e * s.R + j] = sum;
            if (IN_LDS) cur[e] = sum;
            mine = sum > mine ? sum : mine;
        }
        __syncthreads(); // plane j complete (LDS, or global memory written by this workgroup)
    }
    // exclusive prefix over N' = N_lo..N_hi of the filtered list lengths C(p, N', f+1)
    for (int i = threadIdx.x; i < len; i += blockDim.x)
        s_dyn[i] = s.cnt[((long long)(s.N_lo + i) * QQ + s.Q) * s.R + s.p];
    __syncthreads();
    if (threadIdx.x == 0) {
        long long run = 0;
        for (int i = 0; i < len; ++i) {
            const long long c = s_dyn[i];
            s_dyn[i] = run;
            run = sat_add(run, c);
        }
        s_dyn[len] = run;
        *status = run >= kSat ? OOB_EOVERFLOW : OOB_OK;
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= len; i += blockDim.x) offsets[i] = s_dyn[i];
    // While every count is below 2^32 a second copy of the table in 32 bits halves what a lane
    // reads per comparison step (the reads bound the enumeration kernel); padding stays maximal.
    atomicMax(&s_max, (unsigned long long)mine);
    __syncthreads();
    const bool narrow = s_max < (1ull << 32) && !keep_wide;
    if (narrow)
        for (long long e = threadIdx.x; e < (long long)plane * s.R; e += blockDim.x) {
            const long long v = s.cnt[e];
            s.cnt32[e] = v == 0x7FFFFFFFFFFFFFFFll ? 0xFFFFFFFFu : (unsigned)v;
        }
    if (threadIdx.x == 0) *s.narrow = narrow;
}

// The same counts where kGroup planes fit the LDS together (about 2 400 pairs (N', q); 1 290 at 128 nodes, f = 8).
//
// What bounds it: one workgroup's instructions and the lines that its stores touch.  Written plane by plane a count
// is a line of its own, and the 32-bit copy was a further pass that waited for a read of memory per 1 024 counts; here
// kGroup planes are kept and written as whole pieces of their rows.  The pair (N', q) of a thread's entries comes
// from one division per thread instead of one per entry and plane.  The planes are counted in 32 bits with
// saturating additions first; from the first group of planes that saturates (the first of all where the 64-bit table
// is asked for) they are counted in 64 bits.  (A second pass over all planes from the start: 190 us for the 150
// sizes 1..150, f = 3, up to 128 nodes, whose last planes outgrow 32 bits; 104 us here; two planes at a time in 64 bits 113 us.)  The loop over
// the planes of a group has no exit of its own: with one the 57 sizes 8..64 take 47 us in place of 43.4.
// 56 sizes of 8..64 from a list, f = 8, up to 128 nodes: 43 us, 59 us with 64 bits throughout; counting and listing
// 217 -> 150 us as a caller sees them.  29 sizes 4..32, f = 4: 16 us, 21 us with 64 bits.
constexpr size_t kRingLdsBytes = 152 * 1024; // beside 4 KB of sizes, of the 160 KB of a compute unit
constexpr int kCountThreads = 1024;
static_assert(kGroup == 8, "a row's piece is stored as two or four vectors");

// Two terms more, saturating: at 2^32 - 1, or at 2^62 (three numbers up to 2^62 stay below 2^64).
__device__ __forceinline__ unsigned add_terms(unsigned sum, unsigned a, unsigned b) {
    return __builtin_elementwise_add_sat(__builtin_elementwise_add_sat(sum, a), b);
}
__device__ __forceinline__ unsigned long long add_terms(unsigned long long sum, unsigned long long a, unsigned long long b) {
    const unsigned long long c = sum + a + b;
    return c > (unsigned long long)kSat ? (unsigned long long)kSat : c;
}

// The planes from the group that starts with plane `first` on, in CT; the plane before them is in the ring, the last one
// stays there.  In 32 bits it ends after a group with a count that does not fit, sets *top to it and returns the group's
// first plane, else p + 1; in 64 bits *top is raised to the largest count (of the last plane: no plane before holds a
// larger one).  Called and left by the whole workgroup.
template <typename CT> __device__ int count_planes(const Spec &s, CT *ring, const int *size, int first, CT *top) {
    const int QQ = s.Q + 1, plane = (s.N_hi + 1) * QQ;
    const int N0 = (int)threadIdx.x / QQ, q0 = (int)threadIdx.x - N0 * QQ;
    const int dN = kCountThreads / QQ, dq = kCountThreads - dN * QQ; // from one entry of a thread to its next
    CT mine = 0;
    for (int base = first; base <= s.p; base += kGroup) {
        const int last = s.p - base < kGroup - 1 ? s.p - base : kGroup - 1;
        for (int slot = base > 0 ? 0 : 1; slot <= last; ++slot) {
            const int j = base + slot, n = size[j - 1], nq = n * QQ;
            const CT *prev = ring + ((slot - 1) & (kGroup - 1)) * plane;
            CT *cur = ring + slot * plane;
            int N = N0, q = q0;
            for (int e = threadIdx.x; e < plane; e += kCountThreads) {
                CT sum = 0;
                int Ni = N, qi = q, at = e; // at = Ni * QQ + qi
                for (;;) {
                    const bool two = Ni >= n;
                    const int second = two ? at - nq - (qi > 0) : at;
                    const CT c0 = prev[at], c1 = prev[second];
                    sum = add_terms(sum, c0, two ? c1 : (CT)0);
                    if (Ni - n < n) break;
                    Ni -= 2 * n;
                    at = second - nq - (qi > 1);
                    qi = qi > 2 ? qi - 2 : 0;
                }
                cur[e] = sum;
                if (sizeof(CT) == 8 && j == s.p) mine = sum > mine ? sum : mine;
                N += dN; q += dq;
                if (q >= QQ) { q -= QQ; ++N; }
            }
            __syncthreads(); // plane j complete
        }
        // the group's planes; what follows in a row compares greater than any list position (slots past `last` hold older
        // planes or nothing: read, not used)
        if constexpr (sizeof(CT) == 4) {
            unsigned most = 0; // no plane before holds a larger count than the last one
            for (int i = threadIdx.x; i < plane * 2; i += kCountThreads) {
                const int e = i >> 1, k = (i & 1) * 4;
                const CT *c = ring + k * plane + e;
                uint4 v = make_uint4(c[0], c[plane], c[2 * plane], c[3 * plane]);
                const unsigned at = last - k == 0 ? v.x : last - k == 1 ? v.y : last - k == 2 ? v.z : last - k == 3 ? v.w : 0;
                most = at > most ? at : most;
                v.x = k <= last ? v.x : 0xFFFFFFFFu;
                v.y = k + 1 <= last ? v.y : 0xFFFFFFFFu;
                v.z = k + 2 <= last ? v.z : 0xFFFFFFFFu;
                v.w = k + 3 <= last ? v.w : 0xFFFFFFFFu;
                *reinterpret_cast<uint4 *>(s.cnt32 + (long long)e * s.R + base + k) = v;
            }
            if (most == 0xFFFFFFFFu) *top = most; // (every writer the same)
        } else {
            for (int i = threadIdx.x; i < plane * 4; i += kCountThreads) {
                const int e = i >> 2, k = (i & 3) * 2;
                const CT c0 = ring[k * plane + e], c1 = ring[(k + 1) * plane + e];
                const bool in0 = k <= last, in1 = k + 1 <= last;
                const long long row = (long long)e * s.R + base + k;
                *reinterpret_cast<ulonglong2 *>(s.cnt + row) =
                    make_ulonglong2(in0 ? c0 : 0x7FFFFFFFFFFFFFFFull, in1 ? c1 : 0x7FFFFFFFFFFFFFFFull);
                *reinterpret_cast<uint2 *>(s.cnt32 + row) = make_uint2(in0 ? (unsigned)c0 : 0xFFFFFFFFu, in1 ? (unsigned)c1 : 0xFFFFFFFFu);
            }
        }
        __syncthreads(); // the next plane overwrites the first slot
        if (sizeof(CT) == 4 && *top == (CT)~(CT)0) return base; // uniform
    }
    if (sizeof(CT) == 8) {
        atomicMax(top, mine);
        __syncthreads();
    }
    return s.p + 1;
}

// Exclusive prefix over N' = N_lo..N_hi of the filtered list lengths C(p, N', f+1), at whole[N' * stride], by one wave.
template <typename CT> __device__ void write_offsets(const Spec &s, const CT *whole, int stride, long long *offsets, int *status) {
    const int len = s.N_hi - s.N_lo + 1, lane = threadIdx.x;
    long long run = 0;
    for (int i0 = 0; i0 < len; i0 += 64) {
        const int i = i0 + lane;
        long long v = i < len ? (long long)whole[(s.N_lo + i) * stride] : 0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const long long u = __shfl_up(v, d, 64);
            v = lane >= d ? sat_add(v, u) : v;
        }
        const long long before = __shfl_up(v, 1, 64);
        if (i < len) offsets[i] = lane ? sat_add(run, before) : run;
        run = sat_add(run, __shfl(v, 63, 64));
    }
    if (lane == 0) {
        offsets[len] = run;
        *status = run >= kSat ? OOB_EOVERFLOW : OOB_OK;
    }
}

// Inclusive scan over a wave; lanes without a source add zero (the form that becomes one addition with a lane move).
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned moved(unsigned v) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS> __device__ __forceinline__ float moved(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS> __device__ __forceinline__ double moved(double v) {
    return __hiloint2double((int)moved<CTRL, ROWS>((unsigned)__double2hiint(v)), (int)moved<CTRL, ROWS>((unsigned)__double2loint(v)));
}
template <int N, typename T> __device__ __forceinline__ void scan_lanes(T (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += moved<0x111, 0xf>(v[i]); // row_shr 1, 2, 4, 8
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += moved<0x112, 0xf>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += moved<0x114, 0xf>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += moved<0x118, 0xf>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += moved<0x142, 0xa>(v[i]); // lane 15 of a row to the row behind it
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += moved<0x143, 0xc>(v[i]); // lane 31 to the upper half
}

// The table in 32 bits by node counts instead of by sizes.  For one (N', q) the counts of all j are the running sums of
// C(j, N' - n_{j-1}, max(q-1, 0)), so with j along the lanes a row is one scan of a wave, and it leaves as whole lines; and as many
// node counts as the smallest size has nodes do not depend on each other.  A wave takes a few q's (a chunk) of one node count, one
// barrier for all of a step.  Of size n the last n node counts are needed: they are kept in LDS, with room for a step's own.  An unfiltered
// count (q = 0) is the largest of its row; it is carried in floating point too, which tells in the end whether 32 bits held
// everything (a hundredth of the range is left for rounding: at most p + N' additions of relative error 2^-24).
//
// What bounds it: the chain of N_hi / side steps, each some hundred instructions of a wave, a read of LDS and a barrier: 0.4 us where
// a SIMD has one wave, 0.7 us where it has four; 6 us for the launch and what stands before and after the steps.  As a
// caller sees it, planes one after the other -> here: 57 sizes 8..64, f = 8, up to 128 nodes 43 -> 19 us (25 with a wave for all q's of a
// node count), 63 sizes 2..64, f = 8 40 -> 25 us, 29 sizes 4..32, f = 4 14.5 -> 12.2 us.
constexpr int kScanChunk = 6;          // most q's of a wave
constexpr float kFits = 4252017623.0f; // 0.99 * 2^32
constexpr int kCountWaves = kCountThreads / 64;
// Whether the scans are faster than the planes.  A step of the scans takes about as long as a plane of count_planes; there are N_hi / side
// steps and p planes, and the scans take longer to set up.  Planes of fewer than 512 counts leave most threads without work and pass
// faster.  Planes and scans: 28 sizes 3..30, 45 nodes (15 steps) 14.5 and 12.7 us, 39 sizes 2..40, 48 nodes (24 steps)
// 18.8 and 16.9 us; but 15 sizes 2..16, 22 nodes (11 steps) 7.7 and 11.4 us, 40 sizes 1..40, 48 nodes (48 steps) 22.0 and 28.9 us.
// Below 512 counts, f = 0: 13 sizes 12..24, 24 nodes (2 steps) 5.9 and 7.5 us, 16 sizes 8..24 (3 steps) 7.1 and 7.7 us.  Of 1 300 specifications
// of up to 64 sizes with f up to 20 the scans are slower for seven by this line (5 % at most; six of them outgrow 32 bits), for 115 with 10 throughout.
__host__ __device__ inline bool scans_pay(int p, int N_hi, int QQ, int side) { return p >= ((N_hi + 1) * QQ < 512 ? 16 : 10) + N_hi / side; }

// Where the kept counts are.  A row: C(., N', 0) once more, C(., N', q) for the q's of all chunks, the first in floating point.
struct Scan {
    int chunk, chunks, side, row; // q's of a chunk; chunks; node counts of a step; words of a row (odd: neighbours in other banks)
    int base, len;                // of this lane's size: its first row, its rows (0: a lane without a size)
    int need, none;               // words in all; the row of zeros that a lane without a size reads, the next one it writes
};
// False: does not apply.  Called by whole waves, the same result in all.
__device__ bool scan_layout(const Spec &s, const int *size, int words, Scan *sc) {
    const int lane = threadIdx.x & 63, QQ = s.Q + 1;
    if (s.p > 63) return false;
    sc->chunks = (QQ + kScanChunk - 1) / kScanChunk;
    if (sc->chunks > kCountWaves) return false;
    sc->side = kCountWaves / sc->chunks < size[0] ? kCountWaves / sc->chunks : size[0];
    if (!scans_pay(s.p, s.N_hi, QQ, sc->side)) return false;
    sc->chunk = (QQ + sc->chunks - 1) / sc->chunks;
    sc->row = (sc->chunk * sc->chunks + 2) | 1;
    const int n = lane >= 1 && lane <= s.p ? size[lane - 1] : 0;
    sc->len = n ? (n < s.N_hi + 1 ? n : s.N_hi + 1) + sc->side : 0;
    unsigned upto[1] = {(unsigned)sc->len}; // at most 63 * (1215 + 16) in all
    scan_lanes(upto);
    const int rows = __builtin_amdgcn_readlane((int)upto[0], 63);
    sc->none = rows * sc->row;
    sc->base = sc->len ? ((int)upto[0] - sc->len) * sc->row : sc->none;
    sc->need = (rows + 2) * sc->row + s.N_hi + 1;
    return sc->need <= words;
}

// Called by the whole workgroup.
template <int CH> __device__ float scan_steps(const Spec &s, unsigned *lds, unsigned *whole, const Scan &sc) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int QQ = s.Q + 1, mine = wave % sc.side, q0 = wave / sc.side * CH;
    const bool works = q0 < QQ, full = q0 + CH <= QQ; // wave / side < chunks is q0 < QQ
    // words of this lane's rows, of the row of N' and of the row of N' - n (n is len - side), and what a step adds
    const int words = sc.len ? sc.len * sc.row : 1, step = sc.len ? sc.side * sc.row : 0;
    int put = sc.len ? mine * sc.row : 0, get = put + step >= words ? put + step - words : put + step;
    const unsigned *const from = lds + sc.base + q0;
    unsigned *const to = lds + (sc.len ? sc.base : sc.none + sc.row) + q0;
    const bool last = lane == s.p, past = lane > s.p;
    unsigned *out = s.cnt32 + (mine * QQ + q0) * s.R; // at most 2 432 rows of 64 counts
    float most = 0;
    for (int N0 = 0; N0 <= s.N_hi; N0 += sc.side) {
        const int N = N0 + mine;
        if (works && N <= s.N_hi) {
            unsigned v[CH];
            float f[1] = {0};
#pragma unroll
            for (int i = 0; i < CH; ++i) v[i] = from[get + i];
            if (q0 == 0) {
                f[0] = __uint_as_float(from[get + sc.row - 1]);
                if (N == 0) { // C(0, 0, 0) = 1
                    v[0] = lane == 0 ? 1u : v[0];
                    f[0] = lane == 0 ? 1.0f : f[0];
                }
            }
            scan_lanes(v);
#pragma unroll
            for (int i = 0; i < CH; ++i) to[put + i + 1] = v[i];
            if (q0 == 0) {
                to[put] = v[0];
                scan_lanes(f);
                to[put + sc.row - 1] = __float_as_uint(f[0]);
                most = fmaxf(most, f[0]);
            }
            if (q0 + CH >= QQ && last)
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    if (q0 + i == s.Q) whole[N] = v[i];
            if (lane < s.R) {
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    if (full || q0 + i < QQ) out[(unsigned)(i * s.R + lane)] = past ? 0xFFFFFFFFu : v[i];
            }
        }
        out += sc.side * QQ * s.R;
        put = put + step >= words ? put + step - words : put + step;
        get = get + step >= words ? get + step - words : get + step;
        __syncthreads();
    }
    return most;
}

// write_offsets where no count reaches 2^32: the sums stay exact in double precision, and nothing saturates.
__device__ void write_narrow_offsets(const Spec &s, const unsigned *whole, long long *offsets, int *status) {
    const int len = s.N_hi - s.N_lo + 1, lane = threadIdx.x;
    double run = 0;
    for (int i0 = 0; i0 < len; i0 += 64) {
        const int i = i0 + lane;
        const double own = i < len ? (double)whole[s.N_lo + i] : 0.0;
        double v[1] = {own};
        scan_lanes(v);
        if (i < len) offsets[i] = (long long)(run + (v[0] - own));
        run += __builtin_bit_cast(double, ((unsigned long long)(unsigned)__builtin_amdgcn_readlane(__double2hiint(v[0]), 63) << 32) |
                                              (unsigned)__builtin_amdgcn_readlane(__double2loint(v[0]), 63));
    }
    if (lane == 0) {
        offsets[len] = (long long)run;
        *status = OOB_OK;
    }
}

// Called by the whole workgroup.  True: the 32-bit table is complete, and `whole` holds C(p, N', f+1).
__device__ bool count_by_scan(const Spec &s, unsigned *lds, unsigned *whole, const Scan &sc, unsigned *top) {
    for (int e = threadIdx.x; e < sc.need; e += kCountThreads) lds[e] = 0;
    __syncthreads();
    const float most = sc.chunk == 2   ? scan_steps<2>(s, lds, whole, sc)
                       : sc.chunk == 3 ? scan_steps<3>(s, lds, whole, sc)
                       : sc.chunk == 4 ? scan_steps<4>(s, lds, whole, sc)
                       : sc.chunk == 5 ? scan_steps<5>(s, lds, whole, sc)
                                       : scan_steps<kScanChunk>(s, lds, whole, sc);
    atomicMax(top, __float_as_uint(most)); // not negative: ordered as integers are
    __syncthreads();
    return __uint_as_float(*top) < kFits;
}
static_assert(kScanChunk == 6, "count_by_scan names every size of a chunk; a Q of at least 1 makes chunks of two or more");

// SCAN: the table may be counted by count_by_scan, if the sizes allow it (which the host does not see where they are a list).
template <bool SCAN> __global__ void __launch_bounds__(kCountThreads) k_inst_count_ring(Spec s, long long *offsets, int *status, int keep_wide, int lds_words) {
    HIP_DYNAMIC_SHARED(unsigned long long, s_ring) // [kGroup][plane]: plane j at slot j % kGroup
    __shared__ int s_size[OOB_INST_MAX_P];
    __shared__ int s_bad;
    __shared__ unsigned long long s_max;
    __shared__ unsigned s_max32, s_maxf;
    if (threadIdx.x == 0) { s_bad = 0; s_max = 0; s_max32 = 0; s_maxf = 0; }
    for (int j = threadIdx.x; j < s.p; j += kCountThreads) s_size[j] = size_of(s, j);
    __syncthreads();
    for (int j = threadIdx.x; j < s.p; j += kCountThreads)
        if (s_size[j] < 1 || (j > 0 && s_size[j] <= s_size[j - 1])) s_bad = 1;
    __syncthreads();
    if (s_bad) { // uniform: every thread leaves here
        const int len = s.N_hi - s.N_lo + 1;
        for (int i = threadIdx.x; i <= len; i += kCountThreads) offsets[i] = 0;
        if (threadIdx.x == 0) { *status = OOB_EINVAL; *s.narrow = 0; }
        return;
    }
    const int plane = (s.N_hi + 1) * (s.Q + 1);
    int base = 0; // of the planes to count in 64 bits
    if (!keep_wide) {
        unsigned *ring = reinterpret_cast<unsigned *>(s_ring);
        if constexpr (SCAN) {
            Scan sc;
            if (scan_layout(s, s_size, lds_words, &sc)) { // uniform
                unsigned *whole = ring + sc.need - (s.N_hi + 1);
                if (count_by_scan(s, ring, whole, sc, &s_maxf)) {
                    if (threadIdx.x < 64) write_narrow_offsets(s, whole, offsets, status);
                    if (threadIdx.x == 0) *s.narrow = 1;
                    return;
                }
                __syncthreads(); // the LDS is used anew
            }
        }
        for (int e = threadIdx.x; e < plane; e += kCountThreads) ring[e] = e == 0 ? 1 : 0; // C(0, ., .)
        __syncthreads();
        base = count_planes(s, ring, s_size, 0, &s_max32);
        if (base > s.p) { // uniform: every count fits
            if (threadIdx.x < 64) write_offsets(s, ring + (s.p & (kGroup - 1)) * plane + s.Q, s.Q + 1, offsets, status);
            if (threadIdx.x == 0) *s.narrow = 1;
            return;
        }
        // the groups before: from the 32-bit table, half a group a thread and step
        const int halves = base / (kGroup / 2);
        for (int i = threadIdx.x; i < plane * halves; i += kCountThreads) {
            const int e = i / halves, k = (i - e * halves) * (kGroup / 2);
            const uint4 v = *reinterpret_cast<const uint4 *>(s.cnt32 + (long long)e * s.R + k);
            ulonglong2 *wide = reinterpret_cast<ulonglong2 *>(s.cnt + (long long)e * s.R + k);
            wide[0] = make_ulonglong2(v.x, v.y);
            wide[1] = make_ulonglong2(v.z, v.w);
        }
    }
    const int before = base > 0 ? kGroup - 1 : 0; // slot of the plane before (of plane 0 itself)
    for (int e = threadIdx.x; e < plane; e += kCountThreads)
        s_ring[before * plane + e] = base > 0 ? s.cnt32[(long long)e * s.R + base - 1] : e == 0 ? 1 : 0;
    __syncthreads();
    count_planes(s, s_ring, s_size, base, &s_max);
    if (threadIdx.x < 64) write_offsets(s, s_ring + (s.p & (kGroup - 1)) * plane + s.Q, s.Q + 1, offsets, status);
    if (threadIdx.x == 0) *s.narrow = s_max < (1ull << 32) && !keep_wide;
}

typedef unsigned short u16x4 __attribute__((ext_vector_type(4), aligned(2))); // rows of the output start at any entry
template <int CTRL> __device__ __forceinline__ unsigned quad(unsigned v) { return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true); }
// The 16-bit counts of four templates of the lane's vector, those of the first in the lowest bits, for those of template lane / 16 of the four
// vectors of lanes 4 (lane % 16) ..: turned in a quad, then sixteen lanes a template, so that a store of the wave is four runs of 128 bytes (with the
// lanes of a template four apart 1 343 380 vectors take 63 us, not 51).
__device__ __forceinline__ u16x4 transposed(unsigned long long v) {
    const int lane = threadIdx.x & 63;
    const unsigned sel = lane & 1 ? 0x03020706u : 0x05040100u;
    unsigned d0 = (unsigned)v, d1 = (unsigned)(v >> 32);
    d0 = __builtin_amdgcn_perm(quad<0xB1>(d0), d0, sel); // templates 0 and 1 of a pair of lanes: the even one has 0 of both, the odd one 1
    d1 = __builtin_amdgcn_perm(quad<0xB1>(d1), d1, sel);
    const bool up = lane & 2;
    const unsigned got = quad<0x4E>(up ? d0 : d1);
    const int from = 4 * (4 * (lane & 15) + (lane >> 4));
    const unsigned lo = __builtin_amdgcn_ds_bpermute(from, (int)(up ? got : d0)), hi = __builtin_amdgcn_ds_bpermute(from, (int)(up ? d1 : got));
    return __builtin_bit_cast(u16x4, (unsigned long long)hi << 32 | lo);
}

// One lane per output vector (grid-stride).  A vector at position rho of the list of (N', q)
// over the first j sizes has its highest non-zero count at the largest i < j with
// C(i, N', q) <= rho (the lists over fewer sizes are prefixes of the list over more); it then
// continues at position rho - C(i, N', q) of (N' - n_i, q - 1) over the first i+1 sizes.  The
// sizes are visited in groups of kGroup from the top: all lanes take the same trip through
// the groups, so the kGroup counts of a group are stored by whole waves (128 contiguous bytes
// per template), and one read of kGroup counts fetches every count a lane must compare with in
// that group.  C is non-decreasing along a row, so halving locates i (no indexed registers), and a
// group whose first count exceeds rho holds no pipeline of this vector.
//
// What bounds it: the chain of a vector's pipelines, a read of a row and some 50 instructions each; 1 343 380 vectors take 41 us
// without the stores and 25 with nothing else.  With the list of N' searched lane by lane, the entries of a row counted, its address
// multiplied out and two bytes a lane and store 56.5 us, here 51 (both for a list of 56 of the sizes; 46 for all 57 by arithmetic).  Group 0 of all rows in LDS (where most pipelines are): 65; four
// consecutive vectors a lane, which go their common way once: 76, some lane of a wave parts early.
template <typename CT> // long long, or unsigned when the counting kernel could narrow the table
__device__ __forceinline__ void unrank_all(const Spec &s, const long long *offsets, unsigned short *x,
                                           long long capacity, long long total) {
    const int len = s.N_hi - s.N_lo + 1, QQ = s.Q + 1;
    const unsigned step = (unsigned)QQ * (unsigned)s.R; // entries a node count takes: below 2^19, all below 2^30
    const long long stride = (long long)gridDim.x * blockDim.x;
    const CT *tab = sizeof(CT) == 4 ? (const CT *)s.cnt32 : (const CT *)s.cnt;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
        // Last N' whose list starts at or before idx.  For the wave's first vector by 64 of the offsets a read, evenly spread over those still
        // in question (one read up to 64 lists, two up to 4 096); mostly it is the others' too, and the lanes past its end halve what is behind it.
        const int lane = threadIdx.x & 63;
        const long long idx0 = idx - lane;
        const bool whole = idx0 + 64 <= total; // of the wave
        unsigned short *to = x + ((s.p - 1) / kGroup * kGroup + (lane >> 4)) * capacity + (idx0 + 4 * (lane & 15));
        int lo = 0;
        if (whole) // (a ballot of all lanes)
            for (int n = len; n > 1;) { // lo .. lo + n - 1
                const int each = (n + 63) >> 6, l = lane * each;
                const int k = 63 - __clzll((long long)__ballot(l < n && offsets[lo + l] <= idx0)); // (the first one does)
                lo += k * each;
                n = each < n - k * each ? each : n - k * each;
            }
        if (lo < len - 1 && offsets[lo + 1] <= idx) {
            int hi = len - 1;
            for (++lo; lo < hi;) {
                const int mid = (lo + hi + 1) >> 1;
                if (offsets[mid] <= idx) lo = mid; else hi = mid - 1;
            }
        }
        int N = s.N_lo + lo, q = s.Q;
        CT rho = (CT)(idx - offsets[lo]);
        unsigned at = (unsigned)N * step + (unsigned)q * (unsigned)s.R; // of (N, q) in the table
        // A group can hold a pipeline only if its first count is <= rho.  The first counts of up to
        // eight groups are read in one go (independent reads), so that the many empty groups of the
        // large sizes cost one round trip together instead of one each.
        int gcov = (s.p - 1) / kGroup + 1; // groups gcov.. have been probed with the current (N, q, rho)
        int gnext = -1;                    // highest probed group that can hold a pipeline
        for (int g = (s.p - 1) / kGroup; g >= 0; --g) {
            const int base = g * kGroup;
            if (g < gcov) {
                const CT *r0 = tab + at;
                CT f[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) f[i] = r0[(g - i > 0 ? g - i : 0) * kGroup];
                gnext = -1;
#pragma unroll
                for (int i = 7; i >= 0; --i)
                    if (g - i >= 0 && f[i] <= rho) gnext = g - i;
                gcov = g - 7 > 0 ? g - 7 : 0;
            }
            int kcap = s.p - 1 - base < kGroup - 1 ? s.p - 1 - base : kGroup - 1; // sizes base..base+kcap may get a pipeline
            unsigned long long xlo = 0, xhi = 0; // kGroup 16-bit counts
            while (g == gnext) {
                const CT *row = tab + at + base;
                CT c[kGroup];
#pragma unroll
                for (int k = 0; k < kGroup; ++k) c[k] = row[k];
#pragma unroll
                for (int k = 0; k < kGroup; ++k) asm volatile("" : "+v"(c[k])); // read whole: not one entry after the choice of the one before
                gcov = g;              // whatever follows changes (N, q, rho): the groups below are probed again
                if (c[0] > rho) break; // nothing (more) in this group
                // The last entry <= rho up to kcap: they are a prefix of the row, so by halving (no indexed registers).
                const bool b2 = c[4] <= rho && kcap >= 4;
                int ks = b2 ? 4 : 0;
                CT ck = b2 ? c[4] : c[0];
                const CT c26 = b2 ? c[6] : c[2];
                const bool b1 = c26 <= rho && kcap >= (ks | 2);
                ks = b1 ? ks | 2 : ks;
                ck = b1 ? c26 : ck;
                const CT c15 = b2 ? c[5] : c[1], c37 = b2 ? c[7] : c[3], codd = b1 ? c37 : c15;
                const bool b0 = codd <= rho && kcap >= (ks | 1);
                ks = b0 ? ks | 1 : ks;
                ck = b0 ? codd : ck;
                const int nk = size_of(s, base + ks); // consecutive sizes: arithmetic; a list: one cached read
                if (nk > N) break; // cannot happen with a consistent table; keeps the loop finite
                rho -= ck;
                N -= nk;
                at -= __umul24((unsigned)nk, step) + (q > 0 ? (unsigned)s.R : 0u);
                q = q > 0 ? q - 1 : 0;
                kcap = ks;
                const unsigned long long one = 1ull << (16 * (ks & 3));
                if (b2) xhi += one; else xlo += one;
            }
            if (whole) {
#pragma unroll
                for (int h = 0; h < kGroup; h += 4) {
                    const u16x4 w = transposed(h ? xhi : xlo);
                    if (base + h + (lane >> 4) < s.p) *(u16x4 *)(to + h * capacity) = w;
                }
                to -= kGroup * capacity;
                continue;
            }
            unsigned short *xr = x + (long long)base * capacity + idx; // row `base` of the output, this lane's column
            if (base + kGroup <= s.p) { // whole group: no per-template test
#pragma unroll
                for (int k = 0; k < kGroup; ++k, xr += capacity)
                    *xr = (unsigned short)((k < 4 ? xlo : xhi) >> (16 * (k & 3)));
            } else {
#pragma unroll
                for (int k = 0; k < kGroup; ++k, xr += capacity)
                    if (base + k < s.p) *xr = (unsigned short)((k < 4 ? xlo : xhi) >> (16 * (k & 3)));
            }
        }
    }
}

__global__ void __launch_bounds__(256) k_inst_unrank(Spec s, const long long *offsets, int *status,
                                                     unsigned short *x, long long capacity) {
    if (*status != OOB_OK) return;
    const long long total = offsets[s.N_hi - s.N_lo + 1];
    if (total > capacity) { // uniform: nothing is written
        if (blockIdx.x == 0 && threadIdx.x == 0) *status = OOB_ECAPACITY;
        return;
    }
    if (*s.narrow) unrank_all<unsigned>(s, offsets, x, capacity, total); // the table's type is known here only
    else unrank_all<long long>(s, offsets, x, capacity, total);
}

static bool args_ok(int p, int N_lo, int N_hi, int f) {
    return p >= 1 && p <= OOB_INST_MAX_P && N_lo >= 0 && N_lo <= N_hi && N_hi <= OOB_INST_MAX_N && f >= 0 &&
           f <= OOB_INST_MAX_F;
}

static size_t wide_bytes(int p, int N_hi, int f) {
    const size_t n = (size_t)(N_hi + 1) * (size_t)(f + 2) * (size_t)row_len(p) * sizeof(long long);
    return (n + 255) & ~(size_t)255;
}
static size_t table_bytes(int p, int N_hi, int f) { // header, 64-bit table, 32-bit table
    return kHeaderBytes + wide_bytes(p, N_hi, f) + wide_bytes(p, N_hi, f) / 2 + 256;
}

static int check_spec(const int32_t *sizes, int p, int n0, int N_lo, int N_hi, int f, void *ws, size_t ws_bytes,
                      int64_t *offsets, int32_t *status, Spec *s) {
    if (!args_ok(p, N_lo, N_hi, f) || !ws || !offsets || !status) return OOB_EINVAL;
    if (!sizes && n0 < 1) return OOB_EINVAL;
    if (((uintptr_t)ws & 255) != 0) return OOB_EINVAL;
    if (ws_bytes < table_bytes(p, N_hi, f)) return OOB_ECAPACITY;
    s->sizes = sizes; s->p = p; s->n0 = n0; s->N_lo = N_lo; s->N_hi = N_hi; s->Q = f + 1;
    s->R = row_len(p);
    s->narrow = (int *)ws;
    s->cnt = (long long *)((char *)ws + kHeaderBytes);
    s->cnt32 = (unsigned *)((char *)ws + kHeaderBytes + wide_bytes(p, N_hi, f));
    return OOB_OK;
}

static std::atomic<int> g_keep_wide{0}; // test hook: never use the 32-bit copy of the table

static int launch_count(const Spec &s, int64_t *offsets, int32_t *status, hipStream_t stream) {
    const int keep_wide = g_keep_wide.load();
    const size_t plane = (size_t)(s.N_hi + 1) * (s.Q + 1) * sizeof(long long);
    const size_t scan = (size_t)(s.N_hi - s.N_lo + 2) * sizeof(long long);
    if (kGroup * plane <= kRingLdsBytes) { // faster wherever it fits, see the kernel
        // as many node counts a step as the smallest size, if it is known, and a wave can have at most (scan_layout)
        // Of a list the host does not know the smallest size.  With four (small planes) or eight the kernel that can do both, whose planes take
        // 0.7 us longer, is launched for nothing less often than with the most a wave can have: of 1 180 lists 129 instead of 299 are
        // slower than plane by plane, all together 20.2, 16.2 and 16.2 ms (planes; sixteen; here).
        const int side = !s.sizes ? s.n0 : (s.N_hi + 1) * (s.Q + 1) < 512 ? 4 : 8;
        const bool by_scan = s.p <= 63 && !keep_wide && scans_pay(s.p, s.N_hi, s.Q + 1, side < kCountWaves ? side : kCountWaves);
        const size_t lds = by_scan ? kRingLdsBytes : kGroup * plane; // one workgroup: the scans may have all there is
        const auto kernel = by_scan ? k_inst_count_ring<true> : k_inst_count_ring<false>;
        if (lds > 48 * 1024 && // with the 4 KB of sizes above what a launch may ask for unannounced
            hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return OOB_EHIP;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kCountThreads), lds, stream, s, (long long *)offsets, status, keep_wide,
                           (int)(lds / sizeof(unsigned)));
    } else if (2 * plane <= 128 * 1024) {
        const size_t lds = 2 * plane > scan ? 2 * plane : scan;
        if (lds > 48 * 1024 && // (as above)
            hipFuncSetAttribute((const void *)k_inst_count<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return OOB_EHIP;
        hipLaunchKernelGGL(k_inst_count<true>, dim3(1), dim3(1024), lds, stream, s, (long long *)offsets, status,
                           keep_wide);
    } else {
        hipLaunchKernelGGL(k_inst_count<false>, dim3(1), dim3(1024), scan, stream, s, (long long *)offsets, status,
                           keep_wide);
    }
    return hipGetLastError() == hipSuccess ? OOB_OK : OOB_EHIP;
}

static int launch_unrank(const Spec &s, const int64_t *offsets, int32_t *status, uint16_t *x, int64_t capacity,
                         hipStream_t stream) {
    // one lane per vector of the capacity; the kernel strides if the grid limit cuts that short
    const long long want = (capacity + 255) / 256;
    const int grid = (int)(want < 1 ? 1 : (want > (1 << 22) ? (1 << 22) : want));
    hipLaunchKernelGGL(k_inst_unrank, dim3(grid), dim3(256), 0, stream, s, (const long long *)offsets, status,
                       (unsigned short *)x, (long long)capacity);
    return hipGetLastError() == hipSuccess ? OOB_OK : OOB_EHIP;
}

// The count table of oob_inst_enumerate_static: one array per GPU, part of the loaded code object
// (so nothing is ever allocated for it), held until the process ends.  `scratch` itself is a
// host-side stand-in, not a device address: host code uses the address hipGetSymbolAddress reports
// for the current device, looked up once per device.
static __device__ __align__(256) unsigned char scratch[OOB_INST_STATIC_BYTES];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices];

static int static_table(void **ws) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return OOB_EHIP;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return OOB_EHIP;
        }
        g_scratch_ptr[dev] = ptr;
    }
    *ws = g_scratch_ptr[dev];
    return OOB_OK;
}

} // namespace oob_inst

extern "C" {

int oob_inst_keep_wide_table(int on) { return oob_inst::g_keep_wide.exchange(on != 0); }

size_t oob_inst_workspace_size(int p, int N_hi, int f) {
    if (!oob_inst::args_ok(p, 0, N_hi, f)) return 0;
    return oob_inst::table_bytes(p, N_hi, f);
}

int oob_inst_count(const int32_t *sizes, int p, int n0, int N_lo, int N_hi, int f, void *dev_workspace,
                   size_t workspace_bytes, int64_t *offsets, int32_t *status, void *stream) {
    using namespace oob_inst;
    Spec s;
    const int rc = check_spec(sizes, p, n0, N_lo, N_hi, f, dev_workspace, workspace_bytes, offsets, status, &s);
    if (rc != OOB_OK) return rc;
    return launch_count(s, offsets, status, (hipStream_t)stream);
}

int oob_inst_enumerate(const int32_t *sizes, int p, int n0, int N_lo, int N_hi, int f, void *dev_workspace,
                       size_t workspace_bytes, uint16_t *x, int64_t capacity, const int64_t *offsets,
                       int32_t *status, void *stream) {
    using namespace oob_inst;
    Spec s;
    const int rc = check_spec(sizes, p, n0, N_lo, N_hi, f, dev_workspace, workspace_bytes, (int64_t *)offsets,
                              status, &s);
    if (rc != OOB_OK) return rc;
    if (capacity < 0 || (capacity > 0 && !x)) return OOB_EINVAL;
    return launch_unrank(s, offsets, status, x, capacity, (hipStream_t)stream);
}

int oob_inst_enumerate_static(const int32_t *sizes, int p, int n0, int N_lo, int N_hi, int f, uint16_t *x,
                              int64_t capacity, int64_t *offsets, int32_t *status, void *stream) {
    using namespace oob_inst;
    if (!args_ok(p, N_lo, N_hi, f) || !offsets || !status || (!sizes && n0 < 1)) return OOB_EINVAL;
    if (capacity < 0 || (capacity > 0 && !x)) return OOB_EINVAL;
    if (table_bytes(p, N_hi, f) > OOB_INST_STATIC_BYTES) return OOB_ECAPACITY;
    void *ws = nullptr;
    const int rs = static_table(&ws);
    if (rs != OOB_OK) return rs;
    Spec s;
    const int rc = check_spec(sizes, p, n0, N_lo, N_hi, f, ws, OOB_INST_STATIC_BYTES, offsets, status, &s);
    if (rc != OOB_OK) return rc;
    // every entry of the table that is read is written by the counting kernel first: nothing of the
    // previous call's contents survives into this one, and nothing has to be cleared
    const int rl = launch_count(s, offsets, status, (hipStream_t)stream);
    if (rl != OOB_OK) return rl;
    return launch_unrank(s, offsets, status, x, capacity, (hipStream_t)stream);
}

} // extern "C"
