// Spatially ordered dominance path (internal): the points are put in an order
// in which 128 consecutive ones are neighbours in objective space, so that
// most pairs of 128-point blocks are decided by their bounding boxes and only
// the rest are probed (N = 200k, M = 5: 9 % of the pairs, in 3.2 of the 5
// objectives; in the key-sum order half of all pairs, in every objective).
// The dominator masks those probes find are kept, and the front of every
// point is read off them level by level.
//
//   order   quantile cells of the objectives (bit-interleaved), points of a
//           cell in lexicographic key order: identical rows are adjacent
//   tables  128-member tables (bitdom_wide.h) and the box of every block
//   pairs   the dominators of every point within every block that may hold
//           some: degrees, and the masks kept for the ranks
//   ranks   one persistent launch walks the levels of Eq. (8)-(9)
//
// The points of a large problem lie in few fronts, and a level costs as much
// as its unranked points have stored masks.  There the first fronts are taken
// off whole: a pass for the degrees gives front 0 (nobody dominates it), the
// others are copied together in order, the next pass over them gives front 1,
// and so on, as long as a front holds a tenth of the points; masks are stored in
// the last pass only, for what is left.
//
// Whole selections, key-sum order -> this path (with the stages after it as
// they are now): N = 200k, M = 5 2.65 -> 1.33 ms, N = 100k, M = 10 0.95 -> 0.55 ms,
// N = 50k, M = 4 0.74 -> 0.52 ms, N = 20k, M = 3 0.76 -> 0.37 ms, N = 10k, M = 2
// 4.1 -> 0.68 ms, N = 200 0.24 -> 0.075 ms.
#pragma once

#include "bitdom_wide.h"
#include "common.h"

namespace nsga3 {

// Largest problem of this path: the rank launch keeps the unranked set and its
// work-group's rows in LDS, 158,160 of 163,840 B at this size, and the masks grow with
// N * N.  One point more takes the key-sum order and about twice the time (M = 5:
// 1.37 ms here, 2.70 there).
constexpr int64_t kPairsMaxN = 204800;
constexpr int kSplitterSample = 1024;   // keys sampled per objective for the cell splitters
constexpr int kSplitterMaxBits = 6;     // cells per objective: at most 64
constexpr int kCellMaxBits = 16;
constexpr int kHeavyRows = 64;          // rows that are a large share of the points: cells of their own
constexpr int kHeavySample = 16;        // of the sampled rows, at least
constexpr int kHeavyMinN = 4096;        // fewer points count their cells (at most 20 us; finding the
                                        // rows costs every call 2 us)
constexpr int kListItem = 8;            // blocks of a listed pair item
constexpr int kListGroups = 1536;       // work-groups that take them (six a CU)
constexpr int kPairWaves = 4;           // 128-point tiles of a pair work-group (one per wave)
constexpr int kPhaseThreads = 1024;     // positions of a compaction chunk
// Work-groups of the persistent rank launch: 8 waves while one 64-point group a
// wave is enough (N <= 32768; 16 waves took 5 % longer, N = 20k, M = 3 and
// N = 10k, M = 2), 16 for what the phases leave of larger problems.
constexpr int kRankWaves = 8, kRestWaves = 16;
// Work-groups of it, at most (and at most a quarter of the CUs, so that four
// streams' launches run beside each other).  They wait for each other's words,
// and nothing promises that all of them are on the chip at once: other streams'
// kernels, other processes or a CU mask may keep some out.  So those that have
// started form the team (rank_team): it closes when all wanted have started or
// kTeamWait after its first has waited in vain, works through all points with
// as many as it has, and a work-group that starts later leaves.  A team waits
// only for work-groups that are running.  (No measurable time where all start:
// N = 20k, M = 3 370.2 us by block index, 370.5 so; N = 200k, M = 5 1351 / 1352.)
constexpr int kRankMaxGroups = 64;
constexpr uint64_t kTeamWait = 10000;   // ticks of the 100 MHz clock: 100 us
constexpr int kMaxPhases = 5;           // fronts that may be taken off before it

// LDS for the smallest keys of the blocks in the rank launches; a problem with
// more blocks looks at fewer objectives.
constexpr int kRankLowBytes = 32768;


// Stored masks: units of 2 KiB (128 points x 128 members) handed out from
// kMaskPools counters, or from one where there are no more pairs than those (N <=
// 1024: nothing is kept for uneven counters, 1 MiB else).  Up to kMaskFullUnits every pair of blocks has one;
// beyond, half of the pairs up to kMaskHalfUnits units (and for 10 objectives or
// more), then a third.  The masks
// are needed by the pairs whose boxes overlap in some objective and lie in order
// in the others: 10 % of all for sphere-shaped populations, 13-16 % for uniform or
// normal ones, 23 to 36 % where the objectives move together in part, the most for
// few blocks and many objectives.  A pair without a unit is probed again wherever
// a level needs it, which is 30 times a mask's reads: with a sixteenth of the pairs
// the ranks of 200k uniform points, M = 5, took 17 ms instead of 1.3 (the
// workspace 1.7 GB instead of 0.37, which allocate in the same 50 us), and a tenth of
// the pairs without one at N = 60k, M = 16 6.7 ms instead of 0.33.
constexpr int kMaskPools = 64;
constexpr size_t kMaskFullUnits = 16384, kMaskHalfUnits = 524288;
constexpr uint32_t kUnitNone = 0xffffffffu;  // no unit: probe again
inline size_t mask_units(size_t nB, int M) {
    const size_t full = nB * nB;
    size_t u = full / 2 < kMaskHalfUnits || M >= 10 ? full / 2 : kMaskHalfUnits;
    if (u < full / 3) u = full / 3;
    if (u < kMaskFullUnits) u = full < kMaskFullUnits ? full : kMaskFullUnits;
    return full <= kMaskPools ? full : (u + kMaskPools - 1) / kMaskPools * kMaskPools + 8 * kMaskPools;
}

// Counters of the rank launches.
struct alignas(128) RankWord {
    uint64_t v;
    uint64_t pad[15];
};
struct RankSync {
    uint32_t lv[kMaxPhases];     // points of the fronts taken off first
    int32_t left[kMaxPhases];    // points left after each of them
    uint32_t chunk[kMaxPhases][kPairsMaxN / kPhaseThreads];   // the same of a compaction chunk
    uint32_t items[kMaxPhases + 1], next[kMaxPhases + 1];   // listed and taken items of a pass
    RankWord team;               // v [15:0] work-groups that have started, [31:16] the closed
                                 // team's size
    RankWord pool[kMaskPools];   // units taken (v)
};

// One problem: sizes and workspace pointers.
struct PairInst {
    const float *objs;
    int32_t N, M;
    int64_t K;
    int32_t nB;               // 128-point blocks
    int32_t nBpad;            // nB rounded to 64
    int32_t T;                // cell code bits
    int32_t groups;           // work-groups wanted by the persistent rank launch
    int32_t started;          // work-groups it starts (groups, but for tests)
    int32_t rounds;           // 64-point groups of a wave that its LDS holds at once
    int32_t lookPolls;        // looks at a count before a work-group makes it itself
    uint8_t bits[16];         // cell code bits per objective
    uint32_t *spl;            // [M * 64] splitters
    uint32_t *cell;           // [pair_cells(T) + 1] counts, then starts
    uint32_t *heavy;          // number of heavy rows, then hash and keys of each
    uint32_t *code, *slot;    // [N] cell, arrival position in it; code is sval's other buffer
                              // in the phases
    uint32_t *trec;           // [N * rec_stride] records in cell order (keys, point index);
                              // afterwards the other buffer of the phases
    uint32_t *recs;           // [N * rec_stride] records in final order (keys, position)
    uint32_t *sval;           // [N] point index of a position
    int32_t *runs, *rune;     // [N] positions [runs, rune) hold rows identical to this one
    uint32_t *tabs;           // [nB] wide tables
    uint32_t *box;            // [2][M][nBpad] smallest and largest key of a block
    uint64_t *nz;             // [nB][nBpad / 64] blocks whose masks are stored (zeroed)
    uint4 *list;              // items of a pass: kListItem x (block and the tiles that meet it,
                              // objectives to search for each tile, tile group)
    uint32_t *idx;            // [nB][nBpad] mask unit of a stored pair
    uint4 *mask;              // [units + 1][128] dominators of a point within a block; the
                              // last unit is all ones
    uint32_t poolMask;        // pools - 1 (a power of two)
    uint32_t poolUnits;       // units of one pool
    uint32_t allUnit;         // the unit that is all ones
    int32_t *din, *dout;      // [N] degrees in final order (zeroed)
    int32_t *runs2, *rune2, *din2;     // [N] other buffers of the phases
    uint32_t *low;            // [2 * nB][16] smallest keys of the points of a 64-point group
    int32_t lowK;             // objectives whose smallest keys the rank launches look at
    uint64_t *ex;             // [2][M + 2][2 * nBpad] of the unranked points of a 64-point group:
                              // smallest keys, and their set in two halves; [31:0] of a word,
                              // [63:32] the level, double buffered by level (zeroed)
    uint16_t *pos;            // [nB * 128] block of a point's witness
    uint4 *wit;               // [nB * 128] its dominators in that block
    RankSync *sync;           // (zeroed)
    DevScalars *sc;
    int32_t *rank, *dom_in, *dom_out;  // outputs in original order (dom_* may be null)
    uint32_t *tabs64;         // 64-member tables of all points, for a caller that probes them (or null)
};

// Members of a block at positions [lo, hi).
__device__ __forceinline__ void range_bits128(int32_t lo, int32_t hi, uint32_t (&m)[4]) {
    uint32_t a[4], b[4];
    low_bits128((uint32_t)max(lo, 0), a);
    low_bits128((uint32_t)max(hi, 0), b);
#pragma unroll
    for (int q = 0; q < 4; ++q) m[q] = b[q] & ~a[q];
}

// Fronts taken off after `step` phases, and whether no further one is.  A pass for
// one more front costs as much as the last one, which it makes smaller by twice
// the front's share of the points: it pays where that share was a tenth in the
// front before (shells, N = 70k, M = 3: 0.95 ms, with a twentieth 1.03; at N = 200k
// uniform points, M = 5, 3.7 ms with five fronts whatever they hold, 3.25 so,
// normal ones, M = 4, 4.4 and 3.6, shells 1.42 either way).
constexpr uint32_t kPhaseShare = 10;
struct PhaseAt {
    int32_t taken;
    bool stop;
};
__device__ __forceinline__ PhaseAt phase_at(const PairInst &I, int32_t step) {
    if (step == 0) return {0, false};
    uint32_t lv[kMaxPhases], left[kMaxPhases];
#pragma unroll
    for (int q = 0; q < kMaxPhases; ++q) {  // (every load before the first use)
        lv[q] = q < step ? I.sync->lv[q] : 0u;
        left[q] = q < step ? (uint32_t)I.sync->left[q] : 0u;
    }
    PhaseAt a = {0, false};
#pragma unroll
    for (int q = 0; q < kMaxPhases; ++q)
        if (q < step && !a.stop) {
            a.taken = q + 1;
            a.stop = (kPhaseShare - 1u) * lv[q] < left[q];
        }
    return a;
}

// The instance after `taken` fronts: the points left, their number read from the
// device, in the buffers that they went to.
__device__ __forceinline__ PairInst phase_inst(PairInst I, int32_t taken) {
    if (taken == 0) return I;
    I.N = I.sync->left[taken - 1];
    I.nB = (I.N + kWBlk - 1) / kWBlk;
    I.nBpad = (I.nB + 63) / 64 * 64;
    I.dom_in = I.dom_out = nullptr;
    if (taken & 1) {
        I.recs = I.trec;
        I.sval = I.code;
        I.runs = I.runs2;
        I.rune = I.rune2;
        I.din = I.din2;
    }
    return I;
}

// Fronts taken off before the masks are stored, at most: none while one 64-point group
// a wave of the rank launch is enough (N <= 32k).
// Of many objectives the first two fronts hold nearly all points (N = 100k,
// M = 10: one front; three phases more are twelve empty launches, 54 us).
inline int pair_phases(int64_t N, int M) {
    return N <= 32768 ? 0 : N <= 65536 || M >= 8 ? 2 : 5;
}

// Cells of T code bits, and behind them those of the heavy rows.
__host__ __device__ inline int pair_heavy_cell(int T) { return T < 2 ? 4 : 1 << T; }
__host__ __device__ inline int pair_cells(int T) { return pair_heavy_cell(T) + kHeavyRows; }

inline void pair_cell_bits(int64_t N, int M, uint8_t *bits, int *T) {
    int lg = 0;
    while (((int64_t)1 << (lg + 1)) <= N) ++lg;
    int t = lg - 3;
    if (t > kCellMaxBits) t = kCellMaxBits;
    if (t > kSplitterMaxBits * M) t = kSplitterMaxBits * M;
    if (t < 1) t = 1;
    for (int k = 0; k < 16; ++k) bits[k] = (uint8_t)(k < M ? t / M + (k < t % M ? 1 : 0) : 0);
    *T = t;
}

}  // namespace nsga3
