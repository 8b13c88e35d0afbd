// Index arithmetic, LDS and workspace layout of the exact minimum (oob_exact.hip) that the host can check over everything the entry points
// accept: plain C++, so that a CPU test compiles it too.
#pragma once

#include <stddef.h>

#include <initializer_list>

#ifdef __HIPCC__
#define OOB_HD __host__ __device__
#else
#define OOB_HD
#endif

namespace oob_exact {

// i / M for an index i = l M + d of a table with M GPU counts per layer (l <= 255, d < M <= 64) as i recip(M) >> 20.  With
// e = M recip(M) - 2^20 <= M the quotient is i / M + i e / (2^20 M): exact while i e < 2^20, and i e <= (256 M - 1) M < 2^20.
// The product stays below 256 M (2^20 / M + 1) < 2^29.
constexpr int kRecipShift = 20;
OOB_HD inline unsigned recip(int M) { return (1u << kRecipShift) / (unsigned)M + 1; }
OOB_HD inline int quot(int i, unsigned recip_M) { return (int)((unsigned)i * recip_M >> kRecipShift); }

constexpr size_t kLdsLimit = 160 * 1024;
constexpr size_t kLdsStatic = 512;   // left to the kernels' own static arrays
constexpr int kBins = 4096;          // of the order of the list of slowest stages
constexpr size_t kPrepStatic = kBins * sizeof(int) + 1024; // static arrays of k_exact_prep
// Whether a launch with so much dynamic LDS beside static arrays has to be announced (hipFuncAttributeMaxDynamicSharedMemorySize).
inline bool beyond_default(size_t dynamic, size_t fixed) { return dynamic + fixed > 64 * 1024; }
constexpr int kEvalThreads = 512;    // two workgroups per compute unit where LDS allows
constexpr int kStagedThreads = 1024; // with stage counts: one, it needs all the LDS

OOB_HD inline size_t tri(int L) { return (size_t)L * (L + 1) / 2; }
OOB_HD inline int imin(int a, int b) { return a < b ? a : b; }
OOB_HD inline int imax(int a, int b) { return a > b ? a : b; }

// Eight GPUs per node have kernels with the rows of the profile padded to an odd number of doubles: rows of 64 bytes fall on the same
// few banks (63 % of the LDS cycles of the bounds were conflicts, 1 % with rows of nine; 98 layers 780 -> 662 us).
// Other numbers of GPUs have no such kernels: not measured.
OOB_HD inline bool can_pad(int M) { return M == 8; }
// The profile in LDS (see Prof) with rows of ms doubles, in doubles.
OOB_HD inline size_t prof_doubles(int L, int M, int ms, bool sums = false) {
    return (sums ? 1 : 2) * (size_t)(L + 1) * ms + (L + 1) + ((size_t)(L + 1) * M + 7) / 8;
}
// Entries of a band matrix with rows r = 1 .. band and columns 0 .. len - r.
OOB_HD inline size_t band_size(int band, int len) { return (size_t)band * len - (size_t)band * (band - 1) / 2; }

// Tables of k_exact_eval beside its pool: profile, reach, NP, OUT (see Eval) and the minima, in doubles.  No pipeline has
// more nodes than layers.
OOB_HD inline size_t eval_fixed(int L, int M, int n_max, int count, int J, bool sums = false, bool pad = false) {
    const int nodes = imin(n_max, L);
    return prof_doubles(L, M, pad ? M | 1 : M, sums) + ((size_t)(L + 1) * M + 7) / 8 + 2 * (size_t)(L + 2) * J + 2 * (size_t)nodes * M * J + 8 +
           imin(count, nodes);
}
// Its pool for any slowest stage without stage counts, in doubles: the covers next to it, both W and one one-node table,
// bands as wide as the sides are long.
OOB_HD inline size_t eval_pool(int L, int M) { return tri(L) + (size_t)L * M + (size_t)(L + 1) * (M + 1); }

// Threads of k_exact_eval: a wave takes 64 / M start layers at a time, two rounds of them.
inline int eval_threads(int L, int M, bool staged) {
    if (staged) return kStagedThreads;
    int slots = 64, waves = 4;
    while (slots > 1 && 64 / slots < M) slots >>= 1;
    while (waves < kEvalThreads / 64 && waves * slots * 2 < L) waves *= 2;
    return waves * 64;
}
// Whether oob_exact_minimum holds its tables in LDS, as doubles: then no other path follows and the times of a job have to stay
// in the range where doubles are exact.  Status and workspace of a shape follow from it, so the line is a part of
// the interface and stays where the first layout of these tables (two one-node tables, no copy of the profile) filled the LDS.
inline bool in_doubles(int L, int M, int n_max, int count) {
    const size_t row = (size_t)(L + 1) * M;
    return 8 * (tri(L) + row + (row + 1) / 2 + 2 * (size_t)n_max * M + 5 * (size_t)L + (L + 1) / 2 + 5 + count +
                2 * (size_t)(L + 4) * (M + 1) + 8) <= kLdsLimit;
}
// LDS of k_exact_eval.  Without stage counts the tables of any slowest stage fit (0 bytes: they do not, the
// shape takes the general path), at the latest with the ends of the stages added up where they are read; every
// shape of in_doubles() fits.  With stage counts whatever is left for them, entries beyond that take
// the general path one by one.
// The rows of the profile are padded where that costs no workgroup of a compute unit.
struct EvalLds { size_t bytes; bool sums, pad; };
inline EvalLds eval_lds(int L, int M, int n_max, int count, int J, bool staged) {
    if (staged) return {M <= 8 && 8 * eval_fixed(L, M, n_max, count, J) + 48 * 1024 <= kLdsLimit - kLdsStatic ? kLdsLimit - kLdsStatic : 0, false, false};
    for (const bool sums : {false, true}) {
        // as many workgroups per compute unit as the registers allow (sixteen waves) and their tables leave room for: a share
        // less its static arrays is never below what they take
        auto shares = [&](bool pad) {
            const size_t all = (8 * (eval_fixed(L, M, n_max, count, 1, sums, pad) + eval_pool(L, M)) + 15) & ~(size_t)15;
            const size_t most = 1024 / eval_threads(L, M, false), k = kLdsLimit / (all + kLdsStatic);
            return k < most ? k : most;
        };
        const size_t k = shares(false);
        if (k) return {(kLdsLimit / k - kLdsStatic) & ~(size_t)15, sums, !sums && can_pad(M) && shares(true) == k};
    }
    return {0, false, false};
}

// With stage counts: whether the one-node tables are taken in LDS throughout.  Those in registers are more steps one after the other, and
// k_exact_eval<true, 8> spills 200 registers for them, so with eight GPUs per node they lose where LDS has room for a table of every start layer
// beside the covers and both W of any slowest stage, and no wave has two of them to do: 10 layers, 2 nodes 53 and 72 us, 16 layers 109 and 134
// us.  With more start layers than waves only few nodes with few stage counts still gain, whose rows over (GPUs, stages) are short (20 layers, 2 nodes:
// N_b = 8 182 and 198 us, N_b = 11 207 and 198 us; 4 nodes, N_b = 18 303 and 248 us).
// With four GPUs registers are faster at any depth (10 layers 35 and 30 us).
inline bool eval_tables_in_lds(int L, int M, int n_max, int J) {
    const size_t row = (size_t)M * (M + 1) / 2 + 1, tables = (size_t)(L - 1) * row + tri(L - 1) * M + (size_t)(L - 1) * L * row;
    return M == 8 && (L - 1 <= kStagedThreads / 64 || (n_max <= 3 && J <= 10)) && 8 * (eval_fixed(L, M, n_max, n_max, J) + tables) <= kLdsLimit - kLdsStatic;
}

// No bounds for jobs with at most this many (layer pair, GPU count) triples: the bounds, their filter and the second
// evaluation take 70 us or more whatever the job, what evaluating some thousand stages of a short model takes.
constexpr int kDirectMax = 4096;
constexpr int kMaxBuckets = 512;
constexpr int kBucket = 64; // entries whose bounds a workgroup holds at a time
constexpr int kMaxCount = 64;        // templates per job that the bounds are kept for
constexpr int kLambdas = 8, kMus = 8;
// Least entries per bucket (more only where that would exceed kMaxBuckets).  With the lambdas alone a smaller bucket pays:
// its bounds are tighter and the workgroups of 64 leave compute units idle.  How much hangs on the instance (which
// stages are evaluated): timed in turn, 32 against 64, 24 jobs of 34-97 layers 0.93 of the time (0.53 to 1.17), eight of 98
// layers x 8 GPUs 0.97 (0.83 to 1.09); the bounds themselves took 212 instead of 170 us there, with rows of eight doubles.
// With eight mus the bounds are a quarter of the time and it does not (48 layers, limit binding: 3.05 and 3.30 ms).
OOB_HD inline int bucket_least(int multipliers) { return multipliers > kLambdas ? 64 : 32; }

// The workspace: these words, the lists and bounds of layout(), then the tables of k_exact_flat.
struct Head {
    unsigned ncand, bucket, nbuckets, alive, next, done, over, narrow;
};
inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// LDS of k_exact_bounds in doubles.
OOB_HD inline size_t bound_doubles(int L, int M, int mus, bool pad = false) {
    return prof_doubles(L, M, pad ? M | 1 : M) + 2 * (((size_t)(L + 1) * M + 7) / 8) + (size_t)mus * kLambdas * 2 * (L + 1) +
           kBucket * kMaxCount / 2 + 32;
}
inline int bound_mus(int L, int M, bool staged) {
    int mus = staged ? kMus : 1;
    while (mus > 1 && 8 * bound_doubles(L, M, mus) > kLdsLimit - kLdsStatic) --mus;
    return 8 * bound_doubles(L, M, mus) <= kLdsLimit - kLdsStatic ? mus : 0;
}
// The rows of the profile of k_exact_bounds are padded where that costs no workgroup of a compute unit (two of nine waves at most).
inline bool bound_pad(int L, int M, int mus) {
    auto shares = [&](bool pad) { return imin(2, (int)(kLdsLimit / (8 * bound_doubles(L, M, mus, pad) + kLdsStatic))); };
    return can_pad(M) && shares(true) == shares(false);
}
// LDS of k_exact_prep beside its static arrays: bytes, times where the fast path needs them, first layers, and `room` entries of the list.
struct PrepLds { size_t bytes; int room; };
inline PrepLds prep_lds(int L, int M, bool fast) {
    const size_t row = (size_t)(L + 1) * M, tables = 8 * ((size_t)(L + 1) + (fast ? row : 0)) + (row + 3) / 4 * 4;
    const size_t left = kLdsLimit - kPrepStatic - tables, list = 4 * tri(L) * M;
    const int room = fast ? (int)((list < left ? list : left) / 4) : 0;
    return {tables + 4 * (size_t)room, room};
}
struct Layout { size_t head, PT, flo, ctau, cuvd, lb, blo, bfew, blb, barg, list, over, slots; };
inline Layout layout(int L, int M, int n_max, bool fast, int mus, bool staged) { // mus: of the stage limit, 0: no bounds
    const size_t n = fast ? tri(L) * M : 0, cnt = (size_t)imin(n_max, kMaxCount);
    Layout y;
    size_t o = 0;
    y.head = o; o = align_up(o + sizeof(Head));
    y.PT = o;   o = align_up(o + 8 * (size_t)(L + 1) * M);
    y.flo = o;  o = align_up(o + (size_t)(L + 1) * M);
    y.ctau = o; o = align_up(o + 8 * n);
    y.cuvd = o; o = align_up(o + 4 * n);
    y.lb = o;   o = align_up(o + (n > kDirectMax ? 4 * n * kLambdas * mus : 0));
    y.blo = o;  o = align_up(o + 8 * (size_t)kMaxBuckets);
    y.bfew = o; o = align_up(o + 4 * (size_t)kMaxBuckets);
    y.blb = o;  o = align_up(o + 4 * (size_t)kMaxBuckets * cnt);
    y.barg = o; o = align_up(o + 2 * (size_t)kMaxBuckets * cnt);
    y.list = o; o = align_up(o + 4 * n);
    y.over = o; o = align_up(o + (staged ? 4 * n : 0));
    y.slots = o;
    return y;
}

} // namespace oob_exact
