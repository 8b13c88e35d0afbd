// Reconfiguration simulator (Section 5.1 and Appendix B of the Oobleck paper) for gfx950.
//
// One lane runs one failure sequence.  A trajectory's state is small (at most 64 pipeline sizes
// and a 64-bit mask of the list positions still in use), but it is indexed by data.  Up to 16 pipelines
// and 128 nodes the sizes are bytes in registers and every search over the list works on whole
// words (run_single_losses where a step loses one node, run_in_registers for bursts); beyond that (run_in_lds) the sizes live in LDS, one column per lane (sizes[position][lane], 16 bits, as many rows as there are
// starting pipelines), so that the lanes of a wave never share a bank row for the same position,
// and the mask lives in a register pair.  A list position whose pipeline was absorbed keeps size
// 0, so the two loops that run at every step (which pipeline holds the failing node; who can
// lend) walk all positions with a wave-uniform counter and no branch: LDS offsets are the same
// for all lanes and nothing diverges.  Only the rare merge walks the mask.
// Draws are read and trace words written with the trajectory index fastest, so every global
// access of a wave is one contiguous line.  Every loop below ends after at most 64 or `burst`
// rounds for every lane.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "oob_plan.h"
#include "oob_reconf.h"

namespace oob_reconf {

constexpr int kLanes = 256; // trajectories per workgroup
constexpr int kPackedNodes = 128, kPackedWords = 4;
constexpr int kUnroll = 4;  // list positions per round of the two scans; the list is padded with empty ones

struct Args {
    const int *sizes0;
    int c0, n0, n_hi, f;
    const unsigned *draws;
    int steps, burst;
    long long T;
    unsigned *trace;
    int *final_sizes, *summary, *status;
};

// Nodes at the start; -1 where the starting pipelines are no template sizes or too many nodes for 16 bits.
__device__ __forceinline__ long long start_nodes(const Args &a) {
    long long sum = 0;
    for (int i = 0; i < a.c0; ++i) {
        const int s = a.sizes0[i];
        if (s < a.n0 || s > a.n_hi) return -1;
        sum += s;
    }
    return sum <= OOB_RECONF_MAX_NODES ? sum : -1;
}

__device__ __forceinline__ void write_summary(const Args &a, long long t, int survived, int reinst, int borrowed, int merges,
                                              int alive, int nodes, int viol, int stop) {
    int *sm = a.summary + t;
    sm[OOB_RECONF_SURVIVED * a.T] = survived;
    sm[OOB_RECONF_REINSTANTIATED * a.T] = reinst;
    sm[OOB_RECONF_BORROWED * a.T] = borrowed;
    sm[OOB_RECONF_MERGES * a.T] = merges;
    sm[OOB_RECONF_ALIVE * a.T] = alive;
    sm[OOB_RECONF_NODES * a.T] = nodes;
    sm[OOB_RECONF_VIOLATIONS * a.T] = viol;
    sm[OOB_RECONF_STOP * a.T] = stop;
}

// One trajectory with its sizes in LDS: position i at mine[i * kLanes].
__device__ void run_in_lds(const Args &a, long long t, unsigned short *mine) {
    const int rows = (a.c0 + kUnroll - 1) / kUnroll * kUnroll;
    unsigned total = 0;
    for (int i = 0; i < rows; ++i) {
        const int s = i < a.c0 ? a.sizes0[i] : 0;
        mine[i * kLanes] = (unsigned short)s;
        total += (unsigned)s;
    }
    unsigned long long alive = a.c0 == 64 ? ~0ull : (1ull << a.c0) - 1;
    const unsigned need = (unsigned)(a.f + 1) * (unsigned)a.n0; // fewer nodes: training stops
    int stop = OOB_RECONF_STOP_NONE, viol = 0;
    int survived = 0, sum_reinst = 0, sum_borrowed = 0, sum_merges = 0;
    const unsigned *step_draws = a.draws + t;              // this step's first draw of this trajectory
    const long long step_stride = (long long)a.burst * a.T;
    unsigned *word = a.trace ? a.trace + t : nullptr;      // this step's trace word

    for (int step = 0; step < a.steps; ++step, step_draws += step_stride) {
        int reinst = 0, borrowed = 0, merges = 0;
        if (stop == OOB_RECONF_STOP_NONE) {
            // the losses of this step
            unsigned long long affected = 0;
            const unsigned *draw = step_draws;
            for (int b = 0; b < a.burst && total > 0; ++b, draw += a.T) {
                const unsigned r = __umulhi(*draw, total); // floor(draw * total / 2^32) < total
                // The pipeline that holds node r is the number of positions whose running sum of
                // sizes is <= r (absorbed and empty positions add nothing).  It is below c0, since
                // the last running sum is total > r.
                unsigned run = 0;
                int hit = 0;
                for (int i = 0; i < rows; i += kUnroll) {
#pragma unroll
                    for (int e = 0; e < kUnroll; ++e) {
                        run += mine[(i + e) * kLanes];
                        hit += run <= r;
                    }
                }
                mine[hit * kLanes] -= 1;
                affected |= 1ull << hit;
                --total;
            }
            if (total < need) {
                stop = OOB_RECONF_STOP_TOO_FEW_NODES;
            } else {
                // repairs, in list order
                while (affected && stop == OOB_RECONF_STOP_NONE) {
                    const int i = __ffsll((long long)affected) - 1;
                    affected &= affected - 1;
                    if (!((alive >> i) & 1)) continue; // absorbed by an earlier repair
                    int si = mine[i * kLanes];
                    if (si >= a.n0) { ++reinst; continue; }
                    while (si < a.n0) { // borrow from the largest pipeline above n0, first of equals
                        // one max over (size, 63 - position); position i itself is below n0 here
                        unsigned best = 0;
                        for (int k = 0; k < rows; k += kUnroll) {
#pragma unroll
                            for (int e = 0; e < kUnroll; ++e) {
                                const unsigned key = (unsigned)mine[(k + e) * kLanes] << 6 | (unsigned)(63 - k - e);
                                best = key > best ? key : best;
                            }
                        }
                        if ((int)(best >> 6) <= a.n0) break;
                        mine[(63 - (int)(best & 63)) * kLanes] = (unsigned short)((best >> 6) - 1);
                        ++si;
                        ++borrowed;
                    }
                    while (si < a.n0) { // absorb the smallest other pipeline, first of equals
                        int best = 1 << 30, j = -1;
                        for (unsigned long long m = alive & ~(1ull << i); m; m &= m - 1) {
                            const int k = __ffsll((long long)m) - 1;
                            const int s = mine[k * kLanes];
                            if (s < best) { best = s; j = k; }
                        }
                        if (j < 0) { stop = OOB_RECONF_STOP_NO_PARTNER; break; }
                        si += best;
                        mine[j * kLanes] = 0;
                        alive &= ~(1ull << j);
                        ++merges;
                    }
                    mine[i * kLanes] = (unsigned short)si;
                    if (stop == OOB_RECONF_STOP_NONE && si > a.n_hi) viol |= 1;
                }
                if (stop == OOB_RECONF_STOP_NONE) {
                    ++survived;
                    if (__popcll(alive) < a.f + 1) viol |= 2;
                }
            }
            sum_reinst += reinst; sum_borrowed += borrowed; sum_merges += merges;
        }
        if (word) {
            *word = (unsigned)reinst | (unsigned)borrowed << 8 | (unsigned)merges << 16 |
                    (unsigned)__popcll(alive) << 23 | (unsigned)stop << 30;
            word += a.T;
        }
    }

    if (a.final_sizes)
        for (int i = 0; i < a.c0; ++i) a.final_sizes[(long long)i * a.T + t] = mine[i * kLanes];
    write_summary(a, t, survived, sum_reinst, sum_borrowed, sum_merges, __popcll(alive), (int)total, viol, stop);
}

// One trajectory with its sizes in registers: four list positions to a 32-bit word, one byte each, W words.  Needs at
// most kPackedNodes = 128 nodes (a running sum of sizes then fits its byte, and (128 | r) - sum neither borrows
// nor loses its top bit) and at most 4 W starting pipelines.
//
// What bounds it: the vector ALUs (165 instructions a wave and loss: 255 of the 281 us that 2^20 sequences of 29 bursts of two nodes with 13
// pipelines take; 12 bursts of five 312 us).  With the sizes in LDS a step read every position twice from there and the merge walked the list
// position by position: 318 us for 57 losses one by one, which took 258 us here before run_single_losses.
constexpr unsigned kTops = 0x80808080u;
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pk_max(unsigned x, unsigned y) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(u16x2, x), __builtin_bit_cast(u16x2, y)));
}
__device__ __forceinline__ unsigned pk_min(unsigned x, unsigned y) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(u16x2, x), __builtin_bit_cast(u16x2, y)));
}
// Bytes 0, 1 (or 2, 3) of `size` above those of `low` as two 16-bit keys.
__device__ __forceinline__ unsigned keys01(unsigned size, unsigned low) { return __builtin_amdgcn_perm(size, low, 0x05010400u); }
__device__ __forceinline__ unsigned keys23(unsigned size, unsigned low) { return __builtin_amdgcn_perm(size, low, 0x07030602u); }

template <int W> struct Packed {
    unsigned w[W];
    __device__ __forceinline__ int get(int i) const {
        unsigned v = 0; // an OR of masked words: a choice between words becomes a choice between addresses, in scratch memory
#pragma unroll
        for (int k = 0; k < W; ++k) v |= w[k] & (0u - (unsigned)((i >> 2) == k));
        return (int)(v >> ((i & 3) * 8) & 255u);
    }
    __device__ __forceinline__ void set(int i, int value) {
        const unsigned keep = ~(255u << ((i & 3) * 8)), put = (unsigned)value << ((i & 3) * 8);
#pragma unroll
        for (int k = 0; k < W; ++k) w[k] = (i >> 2) == k ? (w[k] & keep) | put : w[k];
    }
};

template <int W> __device__ void run_in_registers(const Args &a, long long t) {
    Packed<W> size, gone; // gone: 255 at positions that are absorbed or were never there, else 0
    unsigned total = 0;
#pragma unroll
    for (int k = 0; k < W; ++k) {
        size.w[k] = 0; gone.w[k] = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int i = 4 * k + b;
            const unsigned s = i < a.c0 ? (unsigned)a.sizes0[i] : 0u;
            size.w[k] |= s << (8 * b);
            gone.w[k] |= i < a.c0 ? 0u : 255u << (8 * b);
            total += s;
        }
    }
    unsigned alive = (1u << a.c0) - 1; // c0 <= 16
    const unsigned need = (unsigned)(a.f + 1) * (unsigned)a.n0; // fewer nodes: training stops
    int stop = OOB_RECONF_STOP_NONE, viol = 0;
    int survived = 0, sum_reinst = 0, sum_borrowed = 0, sum_merges = 0;
    const unsigned *draw = a.draws + t;               // the draws of this trajectory, in order
    // A step's trace word is stored and the next draw read at the head of the step that follows: the wait for the draw at its
    // end covers the store too, and both have had a step's time by then.
    unsigned *word = a.trace ? a.trace + t : nullptr; // where the last step's word goes
    unsigned last = 0;
    unsigned first = a.steps > 0 ? *draw : 0;         // this step's first draw, read a step ahead

    for (int step = 0; step < a.steps; ++step) {
        const unsigned *step_draw = draw;
        draw += (long long)a.burst * a.T;
        unsigned next = 0;
        if (step + 1 < a.steps) next = *draw;
        if (step > 0 && word) {
            *word = last;
            word += a.T;
        }
        int reinst = 0, borrowed = 0, merges = 0;
        if (stop == OOB_RECONF_STOP_NONE) {
            // the losses of this step
            unsigned affected = 0;
            for (int b = 0; b < a.burst && total > 0; ++b) {
                const unsigned d = b ? step_draw[(long long)b * a.T] : first;
                const unsigned r = __umulhi(d, total) | 128u; // floor(d * total / 2^32) < total, for the comparison below
                const unsigned rs = __builtin_amdgcn_perm(r, r, 0u);
                // The pipeline that holds node r is the first position whose running sum exceeds r: the lowest set
                // top bit of `over`, words in order.
                unsigned run = 0, below = 0; // running sum of the words before, in every byte; their last byte of `over`
                int hit = 0;
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    unsigned p = size.w[k] + (size.w[k] << 8);
                    p += (p << 16) + run;
                    run = __builtin_amdgcn_perm(p, p, 0x03030303u);
                    const unsigned over = ~(rs - p) & kTops;
                    size.w[k] -= (over & ~(over << 8 | below >> 24)) >> 7;
                    below = over;
                    hit += __popc(over ^ kTops);
                }
                affected |= 1u << hit;
                --total;
            }
            if (total < need) {
                stop = OOB_RECONF_STOP_TOO_FEW_NODES;
            } else {
                // repairs, in list order
                while (affected && stop == OOB_RECONF_STOP_NONE) {
                    const int i = __ffs((int)affected) - 1;
                    affected &= affected - 1;
                    if (!((alive >> i) & 1)) continue; // absorbed by an earlier repair
                    int si = size.get(i);
                    if (si >= a.n0) { ++reinst; continue; }
                    while (si < a.n0) { // borrow from the largest pipeline above n0, first of equals
                        // one max over (size, 255 - position); position i itself is below n0 here
                        unsigned best = 0;
#pragma unroll
                        for (int k = 0; k < W; ++k) {
                            const unsigned low = 0xFCFDFEFFu - 0x04040404u * (unsigned)k;
                            best = pk_max(best, pk_max(keys01(size.w[k], low), keys23(size.w[k], low)));
                        }
                        best = pk_max(best, best >> 16) & 0xFFFFu;
                        if ((int)(best >> 8) <= a.n0) break;
                        const int k = 255 - (int)(best & 255u);
                        const unsigned one = 1u << ((k & 3) * 8);
#pragma unroll
                        for (int x = 0; x < W; ++x) size.w[x] -= (k >> 2) == x ? one : 0u;
                        ++si;
                        ++borrowed;
                    }
                    while (si < a.n0) { // absorb the smallest other pipeline, first of equals
                        // one min over (size, position), 255 for the size of position i and of those that are gone
                        gone.set(i, 255);
                        unsigned best = 0xFFFFFFFFu;
#pragma unroll
                        for (int k = 0; k < W; ++k) {
                            const unsigned low = 0x03020100u + 0x04040404u * (unsigned)k, s = size.w[k] | gone.w[k];
                            best = pk_min(best, pk_min(keys01(s, low), keys23(s, low)));
                        }
                        best = pk_min(best, best >> 16) & 0xFFFFu;
                        gone.set(i, 0);
                        if ((best >> 8) == 255u) { stop = OOB_RECONF_STOP_NO_PARTNER; break; }
                        const int j = (int)(best & 255u);
                        si += (int)(best >> 8);
                        size.set(j, 0);
                        gone.set(j, 255);
                        alive &= ~(1u << j);
                        ++merges;
                    }
                    size.set(i, si);
                    if (stop == OOB_RECONF_STOP_NONE && si > a.n_hi) viol |= 1;
                }
                if (stop == OOB_RECONF_STOP_NONE) {
                    ++survived;
                    if (__popc(alive) < a.f + 1) viol |= 2;
                }
            }
            sum_reinst += reinst; sum_borrowed += borrowed; sum_merges += merges;
        }
        last = (unsigned)reinst | (unsigned)borrowed << 8 | (unsigned)merges << 16 |
               (unsigned)__popc(alive) << 23 | (unsigned)stop << 30;
        first = next;
    }
    if (a.steps > 0 && word) *word = last;

    if (a.final_sizes)
#pragma unroll
        for (int i = 0; i < 4 * W; ++i)
            if (i < a.c0) a.final_sizes[(long long)i * a.T + t] = (int)(size.w[i >> 2] >> (8 * (i & 3)) & 255u);
    write_summary(a, t, survived, sum_reinst, sum_borrowed, sum_merges, __popc(alive), (int)total, viol, stop);
}

// Steps of one node (burst 1), in registers, W words, at most kPackedNodes nodes and 4 W starting pipelines.
//
// What one loss can do is narrow: every pipeline has n0 nodes or more before it.  The pipeline that is hit either keeps
// n0, or takes one node from a lender, so that the lender is the one that loses the node, or, where all have exactly
// n0, absorbs the first other pipeline in the list (all are equally small), once.  So nodes left, pipelines left, the
// steps that merge (nodes left == n0 x pipelines left), the step that stops and every violation are the same for all
// sequences: they are scalars.  A step without a merge takes one node from one list position.
//
// The state is the running sums of the sizes, a byte each: position i in byte i / W of word i % W, so that a size is a byte
// of the difference of two words.  A comparison of all positions with one number is an add (the carry into a
// byte's top bit) per word; gathered into one 32-bit mask (bit 8 (i / W) + 4 + i % W, ascending with i) its lowest set bit
// is the first position in list order, and -bit the positions whose running sum changes.
// The largest size needs no search: it falls by one when the last position that has it loses a node, and is 2 n0 - 1
// after a merge.
//
// What bounds it: the vector ALUs (about 85 instructions a wave and step) and the 8 bytes a step moves, about equally.
// 2^20 sequences of 57 steps with 13 pipelines: 257 us with run_in_registers (176 instructions, its merge among them:
// all lanes merge at the same steps, but it tests lane by lane), 123 us here (4.5 TB/s).  Draws and words by ordinary
// loads and stores 129 us, eight steps a group 139 us.
constexpr int kGroup = 4; // steps whose draws are read, and whose trace words are stored, together

template <int W> struct Sums {
    static constexpr unsigned kOnes = 0x01010101u;
    unsigned p[W];
    // Bit mask of the positions whose top bit is set in word[k] + add.
    static __device__ __forceinline__ unsigned gather(const unsigned (&word)[W], unsigned add) {
        unsigned m = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) m |= ((word[k] + add) >> (3 - k)) & (kTops >> (3 - k));
        return m;
    }
    __device__ __forceinline__ void sizes(unsigned (&d)[W]) const {
        d[0] = p[0] - (p[W - 1] << 8);
#pragma unroll
        for (int k = 1; k < W; ++k) d[k] = p[k] - p[k - 1];
    }
    // One node less at the first position of `from`, a mask of that position and all behind it.
    __device__ __forceinline__ void lose(unsigned from) {
#pragma unroll
        for (int k = 0; k < W; ++k) p[k] -= (from >> (4 + k)) & kOnes;
    }
    __device__ __forceinline__ void add(unsigned where, int nodes) {
#pragma unroll
        for (int k = 0; k < W; ++k) p[k] += ((where >> (4 + k)) & kOnes) * (unsigned)nodes;
    }
};

template <int W> __device__ void run_single_losses(const Args &a, long long nodes) {
    const unsigned n0 = (unsigned)a.n0;
    Sums<W> sum;
    unsigned at_most = 0, alive = 0; // largest size; list positions in use
    {
        unsigned run = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) sum.p[k] = 0;
#pragma unroll
        for (int i = 0; i < 4 * W; ++i) {
            const unsigned s = i < a.c0 ? (unsigned)__builtin_amdgcn_readfirstlane(a.sizes0[i]) : 0u;
            run += s;
            sum.p[i % W] |= run << (8 * (i / W));
            at_most = s > at_most ? s : at_most;
            alive |= i < a.c0 ? 1u << (8 * (i / W) + 4 + i % W) : 0u;
        }
    }
    constexpr unsigned kOnes = Sums<W>::kOnes;
    unsigned total = (unsigned)__builtin_amdgcn_readfirstlane((int)nodes); // <= 128
    unsigned left = (unsigned)a.c0;                               // pipelines left
    const unsigned need = (unsigned)(a.f + 1) * n0;               // fewer nodes: training stops
    const unsigned can_lend = (127u - n0) * kOnes;                // sets the top bit of sizes above n0
    unsigned largest = (128u - at_most) * kOnes;                  // ... of the largest size
    unsigned borrowed = 0;
    int stop = OOB_RECONF_STOP_NONE, survived = 0;

    const long long block = (long long)blockIdx.x * kLanes;       // the same for all lanes, as every row below
    const unsigned *draws = a.draws + block;
    unsigned *trace = a.trace ? a.trace + block : nullptr;
    const int lane = threadIdx.x;
    unsigned draw[kGroup], word[kGroup];
#pragma unroll
    for (int e = 0; e < kGroup; ++e) draw[e] = e < a.steps ? __builtin_nontemporal_load(draws + e * a.T + lane) : 0u;

    // A group's trace words are stored, and the next group's draws read, at the head of the group that follows.
    int step = 0;
    for (; step < a.steps && stop == OOB_RECONF_STOP_NONE; step += kGroup) {
        draws += kGroup * a.T;
        if (step > 0 && trace) {
#pragma unroll
            for (int e = 0; e < kGroup; ++e) __builtin_nontemporal_store(word[e], trace + e * a.T + lane);
            trace += kGroup * a.T;
        }
        unsigned next[kGroup];
#pragma unroll
        for (int e = 0; e < kGroup; ++e)
            next[e] = step + kGroup + e < a.steps ? __builtin_nontemporal_load(draws + e * a.T + lane) : 0u;
#pragma unroll
        for (int e = 0; e < kGroup; ++e) {
            if (step + e < a.steps && stop == OOB_RECONF_STOP_NONE) {
                const unsigned r = __umulhi(draw[e], total); // floor(draw * total / 2^32) < total
                const unsigned c = 127u - r;
                // running sums above r: the pipeline that holds node r and all behind it
                const unsigned over = Sums<W>::gather(sum.p, __builtin_amdgcn_perm(c, c, 0u));
                const unsigned hit = over & (0u - over);
                if (total - 1 < need) { // stops, repairs nothing
                    stop = OOB_RECONF_STOP_TOO_FEW_NODES;
                    sum.lose(over);
                    word[e] = left << 23 | (unsigned)stop << 30;
                } else if (total == left * n0) { // nobody can lend: absorb the first other pipeline
                    const unsigned others = alive & ~hit, other = others & (0u - others);
                    sum.lose(over);
                    sum.add(over ^ (0u - other), other < hit ? -(int)n0 : (int)n0);
                    alive &= ~other;
                    largest = (128u - (2 * n0 - 1)) * kOnes;
                    --left;
                    ++survived;
                    word[e] = 1u << 16 | left << 23;
                } else {
                    unsigned size[W];
                    sum.sizes(size);
                    const bool keeps = (hit & Sums<W>::gather(size, can_lend)) != 0;
                    const unsigned most = Sums<W>::gather(size, largest);
                    const unsigned loser = keeps ? hit : most & (0u - most);
                    sum.lose(0u - loser);
                    largest += (most & ~loser) == 0 ? kOnes : 0u;
                    borrowed += keeps ? 0u : 1u;
                    ++survived;
                    word[e] = (keeps ? 1u : 1u << 8) | left << 23;
                }
                --total;
            } else {
                word[e] = left << 23 | (unsigned)stop << 30;
            }
        }
#pragma unroll
        for (int e = 0; e < kGroup; ++e) draw[e] = next[e];
    }
    // the last group's words, then those of the steps after the stop
    if (a.trace && a.steps > 0) {
        const int done = step - kGroup;
#pragma unroll
        for (int e = 0; e < kGroup; ++e)
            if (done + e < a.steps) __builtin_nontemporal_store(word[e], trace + e * a.T + lane);
        trace += kGroup * a.T;
        const unsigned idle = left << 23 | (unsigned)stop << 30;
        for (; step < a.steps; ++step, trace += a.T) __builtin_nontemporal_store(idle, trace + lane);
    }

    const long long t = block + lane;
    unsigned size[W];
    sum.sizes(size);
    if (a.final_sizes)
#pragma unroll
        for (int i = 0; i < 4 * W; ++i)
            if (i < a.c0) a.final_sizes[(long long)i * a.T + t] = (int)(size[i % W] >> (8 * (i / W)) & 255u);
    const int merges = a.c0 - (int)left;
    const int viol = (merges > 0 && 2 * a.n0 - 1 > a.n_hi ? 1 : 0) | (survived > 0 && (int)left < a.f + 1 ? 2 : 0);
    write_summary(a, t, survived, survived - merges - (int)borrowed, (int)borrowed, merges, (int)left, (int)total, viol, stop);
}

// W: words of packed sizes, 0 for more than 16 starting pipelines.  SINGLE: steps of one node.  The number of nodes is in device memory: a
// list of more than kPackedNodes takes the sizes in LDS, the same branch for every lane.  (One kernel for both kinds of steps: bursts of 2 to
// 10 nodes with 4 pipelines took 2-14 % longer, 100 and 107 us for 2^20 sequences of 19 bursts of two.)
template <int W, bool SINGLE> __global__ void __launch_bounds__(kLanes) k_reconf(Args a) {
    HIP_DYNAMIC_SHARED(unsigned short, sizes) // [rows][kLanes], rows = c0 rounded up to kUnroll
    const long long t = (long long)blockIdx.x * kLanes + threadIdx.x;
    const long long nodes = start_nodes(a);
    const bool ok = nodes >= 0;
    if (t == 0) *a.status = ok ? OOB_OK : OOB_EINVAL;
    if (!ok || t >= a.T) return;
    if constexpr (W > 0) {
        if (nodes <= kPackedNodes) {
            if constexpr (SINGLE) run_single_losses<W>(a, nodes);
            else run_in_registers<W>(a, t);
            return;
        }
    }
    run_in_lds(a, t, sizes + threadIdx.x);
}

template <bool SINGLE> static auto kernel_for(int words) {
    return words == 1 ? k_reconf<1, SINGLE> : words == 2 ? k_reconf<2, SINGLE> : words == 3 ? k_reconf<3, SINGLE>
         : words == kPackedWords ? k_reconf<kPackedWords, SINGLE> : k_reconf<0, false>;
}

} // namespace oob_reconf

extern "C" int oob_reconf_simulate(const int32_t *sizes0, int c0, int n0, int n_hi, int f,
                                   const uint32_t *draws, int steps, int burst, int64_t T,
                                   uint32_t *trace, int32_t *final_sizes, int32_t *summary,
                                   int32_t *status, void *stream) {
    using namespace oob_reconf;
    if (!sizes0 || !summary || !status) return OOB_EINVAL;
    if (c0 < 1 || c0 > OOB_RECONF_MAX_PIPELINES || n0 < 1 || n_hi < n0 || n_hi > OOB_RECONF_MAX_NODES || f < 0)
        return OOB_EINVAL;
    if ((long long)(f + 1) * n0 > OOB_RECONF_MAX_NODES) return OOB_EINVAL;
    if (steps < 0 || burst < 1 || burst > OOB_RECONF_MAX_BURST || T < 1) return OOB_EINVAL;
    if (steps > 0 && !draws) return OOB_EINVAL;
    const long long blocks = (T + kLanes - 1) / kLanes;
    if (blocks > 0x7fffffffll) return OOB_EINVAL;
    Args a;
    a.sizes0 = sizes0; a.c0 = c0; a.n0 = n0; a.n_hi = n_hi; a.f = f;
    a.draws = draws; a.steps = steps; a.burst = burst; a.T = T;
    a.trace = trace; a.final_sizes = final_sizes; a.summary = summary; a.status = status;
    const size_t lds = (size_t)((c0 + kUnroll - 1) / kUnroll * kUnroll) * kLanes * sizeof(unsigned short); // <= 32 KB
    const int words = (c0 + 3) / 4;
    hipLaunchKernelGGL(burst == 1 ? kernel_for<true>(words) : kernel_for<false>(words), dim3((unsigned)blocks), dim3(kLanes), lds, (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? OOB_OK : OOB_EHIP;
}
