// Fronts of the spatially ordered path (see pairs.h): Eq. (8)-(9) level by
// level from the stored dominator masks, and the last admitted front (end of
// Sec. IV-A.1).
#include "kernels.h"
#include "pairs.h"
#include "prims.h"

namespace nsga3 {

// ---------------------------------------------------------------------------
// ranks.  Front 0 are the points without a dominator.  At a later level a
// point whose stored masks still hold an unranked dominator stays; the others
// are the front.  A wave owns groups of 64 points.  Per level it first looks
// at the block where a point last had an unranked dominator (its witness);
// points that lost theirs go through the stored blocks below it downwards, all
// 64 in step, so that a block's masks are one 1 KiB load.  Blocks whose
// unranked points have, in some objective, a smallest key above every such
// point's are passed (N = 50k, M = 5: a point reads 4.5 masks in all, not 17,
// and has one witness on average).  After the first blocks the rest of a row
// is shared among the work-group's waves, a 64-block word each: the rows at
// the far corner of objective space are the longest by far, and 64-point
// groups next to each other go to different work-groups.
//
// Small problems take one work-group, others one persistent launch of several
// in step; the points' state is in registers where a wave owns one
// group.  The unranked sets go from level to level through global memory by
// device-scope stores and loads (one work-group: through LDS); every 64-bit
// word carries its level, so a work-group waits for the words themselves and
// not for a barrier after them (a level of N = 20k, M = 3 9.6 us with flags
// behind the stores).  Who waits is a team of work-groups that have all started
// (see kRankMaxGroups).  Large problems come here without their first fronts
// (see pairs.h).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t agent_ld(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Dominators of the point at position `at` within block a, from the tables
// (a pair whose masks were not stored).  Four objectives' searches go side by
// side: eight dependent reads for them.
template <int M>
__device__ __forceinline__ uint4 probe_again(const PairInst &I, int32_t at, int32_t a) {
    constexpr int MP = rec_stride(M);
    const uint32_t *T = I.tabs + (size_t)a * wblk_stride(M);
    const uint32_t *row = I.recs + (size_t)at * MP;
    uint32_t m[4];
    low_bits128(T[2], m);
#pragma unroll 1
    for (int k0 = 0; k0 < M; k0 += 4) {
        uint32_t x[4];
        int k[4], c[4];  // member keys <= x
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            k[g] = min(k0 + g, M - 1);
            x[g] = row[k[g]];
            c[g] = 0;
        }
#pragma unroll
        for (int st = 64; st >= 1; st >>= 1)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                c[g] += T[wblk_key_slot(k[g], c[g] + st - 1)] <= x[g] ? st : 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (c[g] == 127 && T[wblk_key_slot(k[g], 127)] <= x[g]) c[g] = 128;
#pragma unroll
            for (int q = 0; q < 4; ++q) m[q] &= T[wblk_mask(k[g], q, c[g])];
        }
    }
    uint32_t r[4];
    range_bits128(I.runs[at] - a * kWBlk, I.rune[at] - a * kWBlk, r);
    return make_uint4(m[0] & ~r[0], m[1] & ~r[1], m[2] & ~r[2], m[3] & ~r[3]);
}

// Whether mask m holds an unranked member of block a.
__device__ __forceinline__ bool mask_hits(const uint4 &m, const uint64_t *Ul, int32_t a) {
    const uint4 u = *reinterpret_cast<const uint4 *>(Ul + 2 * a);
    return ((m.x & u.x) | (m.y & u.y) | (m.z & u.z) | (m.w & u.w)) != 0u;
}

// A wave-uniform value in scalar registers.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

// What a rank work-group keeps in LDS; slots are its 64-point groups (round *
// waves + wave).
struct RankLds {
    uint64_t *U;      // [2 * nBpad] unranked points
    uint64_t *blkU;   // [nBpad / 64] blocks with any
    uint64_t *rows;   // [slots][nBpad / 64] stored blocks of the slot's tile
    uint32_t *idx;    // [slots][nBpad] their mask units, where they fit (or null)
    uint64_t *open;   // [slots] points that lost their witness
    uint64_t *left;   // [slots] those that have not found another
    uint32_t *low;    // [lowK][nBpad] smallest keys of a block's unranked points
    uint32_t *half;   // [2 * nBpad][M] the same of a 64-point group (one work-group only)
    uint32_t *xm;     // [slots][M] largest keys of the open points
    uint64_t *hit;    // [slots][64] highest block found with an unranked dominator: [63:32]
                      // 1 + block, [31:0] its mask unit
    int32_t *bound;   // [slots] blocks from here on are done with
    int32_t *list;    // [slots] slots with open points
};

// LDS words for the mask units of a work-group's rows.
constexpr int kRankIdxWords = 12288;

__host__ __device__ inline size_t rank_lds_words(int nBp, int M, int lowK, int slots, int solo,
                                                 RankLds *S, uint32_t *base) {
    size_t c = 0;
    auto take = [&](size_t words) {
        const size_t at = c;
        c += (words + 3) / 4 * 4;
        return at;
    };
    const size_t nW = (size_t)nBp / 64;
    const size_t oU = take(4 * (size_t)nBp), oB = take(2 * nW), oR = take(2 * slots * nW);
    const size_t oO = take(4 * (size_t)slots), oL = take((size_t)lowK * nBp);
    const size_t oH = take(solo ? 2 * (size_t)nBp * M : 0), oX = take((size_t)slots * M);
    const size_t oT = take(128 * (size_t)slots), oN = take(slots), oI = take(slots);
    const bool near = slots * nBp <= kRankIdxWords;
    const size_t oQ = take(near ? (size_t)slots * nBp : 0);
    if (S) {
        S->U = reinterpret_cast<uint64_t *>(base + oU);
        S->blkU = reinterpret_cast<uint64_t *>(base + oB);
        S->rows = reinterpret_cast<uint64_t *>(base + oR);
        S->idx = near ? base + oQ : nullptr;
        S->open = reinterpret_cast<uint64_t *>(base + oO);
        S->left = S->open + slots;
        S->low = base + oL;
        S->half = base + oH;
        S->xm = base + oX;
        S->hit = reinterpret_cast<uint64_t *>(base + oT);
        S->bound = reinterpret_cast<int32_t *>(base + oN);
        S->list = reinterpret_cast<int32_t *>(base + oI);
    }
    return c;
}

// A lane's point of one slot.
template <int M>
struct RankPoint {
    uint32_t x[M];       // keys
    uint4 wit;           // its dominators in block p
    int32_t p;           // block of the witness; blocks from p on hold no other unranked dominator
    uint32_t low;        // lane k: smallest key k of the group's unranked points
    uint32_t i;          // point index
    int32_t din, dout;   // degrees
};

// Mask units of word wd of a slot's row, one a lane.
__device__ __forceinline__ uint32_t row_units(const PairInst &I, const RankLds &S, int32_t slot,
                                              int32_t h, int32_t wd) {
    const int32_t b = wd * 64 + (int32_t)lane_id();
    return S.idx ? S.idx[slot * I.nBpad + b] : I.idx[(size_t)(h >> 1) * I.nBpad + b];
}

// More batches than a word has blocks (a batch may hold a single block).
constexpr int kWholeWord = 1 << 20;

// Goes down the stored blocks of word w below `bound`, until about `most` of
// them are looked at (a batch counts as kAhead),
// for the open lanes of a slot: hit receives 1 + the highest block with an
// unranked dominator (upper half) and its mask unit, open is cleared.  iv:
// mask units of the word's blocks, one a lane.  Returns the block all above
// which are done with.
template <int M>
__device__ __forceinline__ int32_t scan_word(const PairInst &I, const RankLds &S, int32_t h,
                                             const uint64_t *row, const uint32_t *xm, int32_t w,
                                             int32_t bound, int most, uint32_t iv, bool &open,
                                             uint64_t &hit) {
    constexpr int kAhead = 8;  // masks read at once
    const int lane = (int)lane_id();
    const int32_t lim = bound - (w << 6);
    uint64_t t = uniform(row[w] & S.blkU[w]) & (lim >= 64 ? ~0ull : (1ull << lim) - 1ull);
    const uint64_t none = ballot(iv == kUnitNone);
    if (t) {
        bool ok = true;  // the lane's block against the open points
#pragma unroll
        for (int k = 0; k < M; ++k)
            if (k < I.lowK) ok = ok && S.low[k * I.nBpad + (w << 6) + lane] <= xm[k];
        t &= ballot(ok);
    }
    // (everything but the masks and their tests is scalar: a batch is 8 loads
    // and 60 vector instructions)
    const char *mk = reinterpret_cast<const char *>(I.mask);
    const uint32_t mine = (uint32_t)((h & 1) * kWave + lane) * 16u;
    int32_t hb = -1;   // highest block with an unranked dominator of the lane's point
    uint32_t hu = 0;
    while (t && most > 0) {
        int32_t b[kAhead];
        uint32_t u[kAhead];
        uint4 m[kAhead];
        int32_t top = 63 - __builtin_clzll(t);
        if ((none >> top) & 1) {  // not stored: this block alone
            m[0] = probe_again<M>(I, min(h * kWave + lane, I.N - 1), (w << 6) + top);
            t &= ~(1ull << top);
            --most;
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                b[q] = top;
                u[q] = kUnitNone;
                if (q) m[q] = make_uint4(0, 0, 0, 0);
            }
        } else {
            // up to kAhead blocks; a short batch repeats its last one
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                b[q] = top;
                u[q] = (uint32_t)__builtin_amdgcn_readlane((int)iv, top);
                t &= ~(1ull << top);
                const int32_t nx = t ? 63 - __builtin_clzll(t) : top;
                top = (none >> nx) & 1 ? top : nx;
                m[q] = *reinterpret_cast<const uint4 *>(mk + (size_t)u[q] * (16 * kWBlk) + mine);
            }
            most -= kAhead;
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const bool in = open && mask_hits(m[q], S.U, (w << 6) + b[q]);
            hb = in ? b[q] : hb;
            hu = in ? u[q] : hu;
            open = open && !in;
        }
        bound = (w << 6) + b[kAhead - 1];
        if (!ballot(open)) {
            t = 1;  // (bound stays)
            break;
        }
    }
    if (hb >= 0) hit = (uint64_t)(uint32_t)((w << 6) + hb + 1) << 32 | hu;
    return t ? bound : w << 6;
}

// Word of the exchange before level rel: field f (keys, then the set's halves)
// of group h.
template <int M>
__device__ __forceinline__ size_t ex_word(const PairInst &I, int32_t rel, int32_t f, int32_t h) {
    return ((size_t)(rel & 1) * (M + 2) + f) * 2 * I.nBpad + h;
}

// One level for the slots of a work-group; `rounds` slots per wave, at most
// `slots` in all.  Slot q is the 64-point group (q0 + q) * G + g.  Returns the wave's
// number of points of this front.  kKeep: one slot per wave, its state stays
// in P over the levels; else it is read from and written to I.pos and I.wit.
template <int M, int kW, bool kKeep, bool kSolo>
__device__ __forceinline__ uint32_t rank_level(const PairInst &I, int32_t level, int32_t base, int32_t g,
                                               int32_t G, int32_t q0, int32_t rounds, int32_t slots,
                                               const RankLds &S, RankPoint<M> &P, int32_t *s_n) {
    constexpr int MP = rec_stride(M);
    constexpr int kFirst = 8;  // blocks a wave looks at by itself before sharing a row
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = (int)lane_id();
    const int32_t nB = I.nB, nW = I.nBpad / 64, nH = 2 * nB;
    const int32_t rel = level - base;
    uint32_t fresh = 0;
    // front 0 by in-degree, later levels: points that lost their witness
#pragma unroll 1
    for (int r = 0; r < (kKeep ? 1 : rounds); ++r) {
        const int slot = r * kW + w;
        const int32_t h = (q0 + slot) * G + g;
        if (slot >= slots || h >= nH) break;
        const uint64_t un = uniform(S.U[h]);
        uint64_t open_m = 0;
        if (un) {
            const int32_t at = h * kWave + lane;
            const bool mem = ((un >> lane) & 1) != 0;
            if (rel == 0) {
                P.p = nB;
                P.wit = make_uint4(0, 0, 0, 0);
            } else if (!kKeep) {
                P.p = mem ? (int32_t)I.pos[at] : nB;
                P.wit = mem ? I.wit[at] : make_uint4(0, 0, 0, 0);
            }
            if (kKeep && rel == 0) {
                P.i = mem ? I.sval[at] : 0u;
                P.din = mem ? I.din[at] : 1;
                P.dout = mem && I.dom_out ? I.dout[at] : 0;
                P.low = lane < M ? I.low[(size_t)h * 16 + lane] : 0u;
#pragma unroll
                for (int k = 0; k < M; ++k) P.x[k] = mem ? I.recs[(size_t)at * MP + k] : 0xffffffffu;
            }
            bool open;
            if (rel == 0)
                open = mem && (kKeep ? P.din : I.din[at]) == 0;
            else
                open = mem && (P.p >= nB || !mask_hits(P.wit, S.U, P.p));
            open_m = ballot(open);
            if (open_m) {
                S.hit[slot * kWave + lane] = 0ull;
                if (rel > 0) {
                    if (!kKeep) {
#pragma unroll
                        for (int k = 0; k < M; ++k)
                            P.x[k] = mem ? I.recs[(size_t)at * MP + k] : 0xffffffffu;
                    }
#pragma unroll
                    for (int k = 0; k < M; ++k) {
                        const uint32_t x = wave_extreme<true>(open ? P.x[k] : 0u);
                        if (lane == 0) S.xm[slot * M + k] = x;
                    }
                    const int32_t bd = (int32_t)wave_extreme<true>(open ? (uint32_t)P.p : 0u);
                    if (lane == 0) S.bound[slot] = bd;
                }
            }
        }
        if (lane == 0) {
            S.open[slot] = open_m;
            S.left[slot] = open_m;
        }
    }
    if (rel > 0) {
        // a wave's own slots first, a few blocks each, all points in step: most
        // find a witness there
#pragma unroll 1
        for (int r = 0; r < (kKeep ? 1 : rounds); ++r) {
            const int slot = r * kW + w;
            const int32_t h = (q0 + slot) * G + g;
            if (slot >= slots || h >= nH) break;
            const uint64_t om = uniform(S.left[slot]);
            if (!om) continue;
            const uint64_t *row = S.rows + (size_t)slot * nW;
            int32_t bound = uniform(S.bound[slot]);
            int32_t wd = (bound + 63) / 64 - 1;  // the highest word with blocks
            while (wd >= 0 && uniform(row[wd] & S.blkU[wd]) == 0ull) --wd;
            if (wd < 0) continue;
            const uint32_t iv = row_units(I, S, slot, h, wd);
            uint32_t xm[M];
#pragma unroll
            for (int k = 0; k < M; ++k) xm[k] = S.xm[slot * M + k];
            bool open = ((om >> lane) & 1) != 0;
            uint64_t hit = 0;
            bound = scan_word<M>(I, S, h, row, xm, wd, bound, kFirst, iv, open, hit);
            if (hit) S.hit[slot * kWave + lane] = hit;
            const uint64_t still = ballot(open);
            if (lane == 0) {
                S.left[slot] = still;
                S.bound[slot] = bound;
                if (still && bound > 0) S.list[atomicAdd(s_n, 1)] = slot;
            }
        }
        __syncthreads();
        // the rest of the rows, a word at a time over all waves
        const int32_t nE = uniform(*s_n);
#pragma unroll 1
        for (int32_t u = w; u < nE * nW; u += kW) {
            const int32_t slot = uniform(S.list[u % nE]);
            const int32_t wd = nW - 1 - u / nE;
            const int32_t h = (q0 + slot) * G + g;
            const int32_t bound = uniform(S.bound[slot]);
            const uint64_t *row = S.rows + (size_t)slot * nW;
            if (bound <= wd << 6 || uniform(row[wd] & S.blkU[wd]) == 0ull) continue;
            const uint32_t iv = row_units(I, S, slot, h, wd);
            uint32_t xm[M];
#pragma unroll
            for (int k = 0; k < M; ++k) xm[k] = S.xm[slot * M + k];
            bool open = ((uniform(S.left[slot]) >> lane) & 1) != 0;
            uint64_t hit = 0;
            scan_word<M>(I, S, h, row, xm, wd, bound, kWholeWord, iv, open, hit);
            if (hit)
                atomicMax((unsigned long long *)&S.hit[slot * kWave + lane],
                          (unsigned long long)hit);
        }
        __syncthreads();
    }
    // fronts, and the unranked sets of the next level
#pragma unroll 1
    for (int r = 0; r < (kKeep ? 1 : rounds); ++r) {
        const int slot = r * kW + w;
        const int32_t h = (q0 + slot) * G + g;
        if (slot >= slots || h >= nH) break;
        const uint64_t un = uniform(S.U[h]);
        const uint64_t om = uniform(S.open[slot]);
        uint64_t front = 0;
        const int32_t at = h * kWave + lane;
        const bool mem = ((un >> lane) & 1) != 0;
        if (om) {
            const bool open = ((om >> lane) & 1) != 0;
            const uint64_t hit = open ? S.hit[slot * kWave + lane] : 0ull;
            if (hit) {
                const uint32_t u = (uint32_t)hit;
                const int32_t p = (int32_t)(hit >> 32) - 1;
                uint4 wit;
                if (u != kUnitNone)
                    wit = I.mask[(size_t)u * kWBlk + (h & 1) * kWave + lane];
                else
                    wit = probe_again<M>(I, at, p);
                if (kKeep) {
                    P.p = p;
                    P.wit = wit;
                } else {
                    I.pos[at] = (uint16_t)p;
                    I.wit[at] = wit;
                }
            }
            front = ballot(open && !hit);
            if (open && !hit) {
                const uint32_t i = kKeep ? P.i : I.sval[at];
                I.rank[i] = level;
                if (I.dom_in) I.dom_in[i] = kKeep ? P.din : I.din[at];
                if (I.dom_out) I.dom_out[i] = kKeep ? P.dout : I.dout[at];
            }
            fresh += (uint32_t)__popcll(front);
        }
        if (rel == 0 && !kKeep && mem && !((front >> lane) & 1)) {
            I.pos[at] = (uint16_t)nB;
            I.wit[at] = make_uint4(0, 0, 0, 0);
        }
        uint32_t keep_low = 0u;
        if (un) {
            // smallest keys of what stays
            uint32_t low = kKeep ? P.low : 0u;
            if (front) {
                const bool stays = mem && !((front >> lane) & 1);
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const uint32_t x = kKeep ? P.x[k] : I.recs[(size_t)min(at, I.N - 1) * MP + k];
                    const uint32_t l = wave_extreme<false>(stays ? x : 0xffffffffu);
                    if (lane == k) low = l;
                }
                if (kKeep) P.low = low;
            } else if (!kKeep && lane < M) {
                low = rel == 0 ? I.low[(size_t)h * 16 + lane]
                               : (uint32_t)agent_ld(&I.ex[ex_word<M>(I, rel, lane, h)]);
            }
            if (kSolo && lane < M) S.half[h * M + lane] = low;
            keep_low = low;
        }
        if (kSolo) {
            if (lane == 0) S.U[h] = un & ~front;
        } else if (lane < M + 2 && (lane >= M || lane < I.lowK)) {
            const uint64_t u = un & ~front;
            const uint32_t v = lane < M ? keep_low : (uint32_t)(lane == M ? u : u >> 32);
            __hip_atomic_store(&I.ex[ex_word<M>(I, rel + 1, lane, h)],
                               (uint64_t)(uint32_t)(rel + 1) << 32 | v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    return fresh;
}

// The unranked set of the rel-th level into LDS (the first: every point).
// Returns this thread's share of it; s_f is set where a work-group's words never
// came.
template <int M, int kW, bool kSolo>
__device__ __forceinline__ uint32_t load_unranked(const PairInst &I, int32_t rel, const RankLds &S,
                                                  uint32_t &s_f) {
    const int32_t nBp = I.nBpad, nH = 2 * I.nB;
    uint32_t mine = 0;
    for (int32_t h0 = 0; h0 < 2 * nBp; h0 += kW * kWave) {
        const int32_t h = h0 + (int32_t)threadIdx.x;  // a thread takes a 64-point group
        uint64_t u = 0;
        uint32_t z[M];
#pragma unroll
        for (int k = 0; k < M; ++k) z[k] = ~0u;
        if (h < nH) {
            if (rel == 0) {
                const int32_t n = I.N - h * kWave;
                u = n >= kWave ? ~0ull : (n <= 0 ? 0ull : (1ull << n) - 1ull);
            } else if (kSolo) {
                u = S.U[h];
#pragma unroll
                for (int k = 0; k < M; ++k) z[k] = S.half[h * M + k];
            } else {
                const uint64_t *e = I.ex + ex_word<M>(I, rel, 0, h);
                uint32_t spins = 0;
                while (true) {  // (every load before the first use)
                    uint64_t y[M + 2];
                    uint32_t off = 0;
#pragma unroll
                    for (int k = 0; k < M + 2; ++k)
                        y[k] = k >= M || k < I.lowK ? agent_ld(&e[(size_t)k * 2 * nBp])
                                                    : (uint64_t)(uint32_t)rel << 32;
#pragma unroll
                    for (int k = 0; k < M + 2; ++k) off |= (uint32_t)(y[k] >> 32) ^ (uint32_t)rel;
                    u = (uint32_t)y[M] | y[M + 1] << 32;
#pragma unroll
                    for (int k = 0; k < M; ++k) z[k] = (uint32_t)y[k];
                    if (off == 0u) break;
                    if (++spins > (1u << 26)) {  // a work-group never arrived
                        atomicOr(&I.sc->err, (uint32_t)kErrBarrierTimeout);
                        s_f = ~0u;
                        break;
                    }
                }
            }
        }
        if (h < 2 * nBp) {  // (whole waves)
            if (!kSolo || rel == 0) S.U[h] = u;
            if (rel > 0) {  // (front 0 looks at no block)
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const uint32_t v = u ? z[k] : ~0u;
                    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xb1,
                                                                             0xf, 0xf, false);
                    if (k < I.lowK && (h & 1) == 0) S.low[k * nBp + (h >> 1)] = min(v, o);
                }
            }
            uint64_t m = ballot(u != 0ull);
            m = (m | m >> 1) & 0x5555555555555555ull;  // a bit per block, then together
            m = (m | m >> 1) & 0x3333333333333333ull;
            m = (m | m >> 2) & 0x0f0f0f0f0f0f0f0full;
            m = (m | m >> 4) & 0x00ff00ff00ff00ffull;
            m = (m | m >> 8) & 0x0000ffff0000ffffull;
            m = m | m >> 16;
            if (lane_id() == 0) reinterpret_cast<uint32_t *>(S.blkU)[h >> 6] = (uint32_t)m;
            mine += (uint32_t)__popcll(u);
        }
    }
    return mine;
}

// Stored-block rows of the work-group's slots from q0 on.
template <int kW>
__device__ __forceinline__ void load_rows(const PairInst &I, int32_t g, int32_t G, int32_t q0,
                                          int32_t slots, const RankLds &S) {
    const int32_t nW = I.nBpad / 64;
    for (int32_t q = (int32_t)threadIdx.x; q < slots * nW; q += kW * kWave) {
        const int32_t tile = ((q0 + q / nW) * G + g) >> 1;
        S.rows[q] = tile < I.nB ? I.nz[(size_t)tile * nW + q % nW] : 0ull;
    }
    if (S.idx)
        for (int32_t q = (int32_t)threadIdx.x; q < slots * I.nBpad; q += kW * kWave) {
            const int32_t tile = ((q0 + q / I.nBpad) * G + g) >> 1;
            S.idx[q] = tile < I.nB ? I.idx[(size_t)tile * I.nBpad + q % I.nBpad] : 0u;
        }
}

// Points of the fronts before level0.
__device__ __forceinline__ uint32_t rank_done(const PairInst &I, int32_t level0) {
    uint32_t n = 0;
    for (int32_t l = 0; l < level0; ++l) n += I.sync->lv[l];
    return n;
}

// This work-group's number g in the team of the launch and the team's size G (0:
// the team has closed without it).  Every member returns the same size: it is
// the wanted number once that many have started, else what one exchange of the
// word fixed, and later starts do not change those bits.
__device__ __forceinline__ void rank_team(const PairInst &I, int32_t *s_team) {
    if (threadIdx.x == 0) {
        uint32_t *word = reinterpret_cast<uint32_t *>(&I.sync->team.v);
        const uint32_t want = (uint32_t)I.groups;
        const uint32_t old = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t g = old & 0xffffu;
        uint32_t G = 0;
        if (old >> 16 == 0u && g < want) {
            uint32_t v = old + 1u;
            const uint64_t t0 = wall_clock64();
            while (true) {
                G = v >> 16 ? v >> 16 : ((v & 0xffffu) >= want ? want : 0u);
                if (G) break;
                if (wall_clock64() - t0 > kTeamWait) {
                    // (v has no size yet; where another work-group changed the word it is read again)
                    const uint32_t closed = v | v << 16;
                    if (__hip_atomic_compare_exchange_strong(word, &v, closed, __ATOMIC_RELAXED,
                                                             __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT))
                        v = closed;
                    continue;
                }
                __builtin_amdgcn_s_sleep(1);
                v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        s_team[0] = (int32_t)g;
        s_team[1] = (int32_t)G;
    }
    __syncthreads();
}

// Every level from level0 on, for the points that I still holds, by work-group g
// of G.  Without kKeep a wave has any number of slots, I.rounds of them in LDS
// at once.
template <int M, int kW, bool kKeep, bool kSolo>
__device__ __forceinline__ void rank_levels(const PairInst &I, int32_t g, int32_t G, int32_t level0,
                                            uint32_t *dyn, uint32_t *s_new, uint32_t *s_fp,
                                            int32_t *s_np) {
    uint32_t &s_f = *s_fp;
    int32_t &s_n = *s_np;
    const int tid = (int)threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = (int)lane_id();
    const int32_t all = (2 * I.nB + G * kW - 1) / (G * kW);
    const int32_t rounds = kKeep ? 1 : min(all, I.rounds);
    RankLds S;
    rank_lds_words(I.nBpad, M, I.lowK, rounds * kW, kSolo, &S, dyn);
    load_rows<kW>(I, g, G, 0, rounds * kW, S);
    RankPoint<M> P;
    uint32_t done = 0;             // points ranked before this level
    bool found = false;
    auto close = [&](int32_t level, uint32_t f) {  // level `level` has f points
        if (g == 0 && tid == 0) {
            if (!found && (int64_t)done + f >= I.K) {
                found = true;
                I.sc->last_front = level;
                I.sc->last_front_size = (int32_t)f;
                I.sc->n_before = done;
                I.sc->num_from_last = I.K - done;
            }
            I.sc->num_fronts = level + 1;
        }
        done += f;
    };
    const uint32_t total = (uint32_t)I.N + rank_done(I, level0);
    for (int32_t level = 0; level < level0; ++level) {
        const uint32_t f = I.sync->lv[level];
        if (f) close(level, f);
    }
    if (I.N == 0) return;
    if (tid == 0) s_f = 0;
    uint32_t prev = 0;  // points unranked before the last level
    __syncthreads();
    for (int32_t level = level0;; ++level) {
        if (tid == 0) s_n = 0;
        if (!kKeep && all > rounds && level > level0) load_rows<kW>(I, g, G, 0, rounds * kW, S);
        const uint32_t mine = load_unranked<M, kW, kSolo>(I, level - level0, S, s_f);
        if (!kSolo) {
            const uint32_t n = wave_sum(mine);
            if (lane == 0) s_new[w] = n;
        }
        lds_wait();
        __syncthreads();
        if (!kSolo) {
            if (s_f == ~0u) return;
            uint32_t left = 0;
            for (int q = 0; q < kW; ++q) left += s_new[q];
            if (level > level0) {
                close(level - 1, prev - left);
                if (left == 0) return;
                if (left == prev) {  // impossible for a partial order
                    if (tid == 0) atomicOr(&I.sc->err, (uint32_t)kErrInternal);
                    return;
                }
            }
            prev = left;
        }
        uint32_t fresh = 0;
#pragma unroll 1
        for (int32_t r0 = 0; r0 < (kKeep ? 1 : all); r0 += rounds) {
            if (r0 > 0) {
                lds_wait();
                __syncthreads();
                if (tid == 0) s_n = 0;
                load_rows<kW>(I, g, G, r0 * kW, rounds * kW, S);
                lds_wait();
                __syncthreads();
            }
            fresh = rank_level<M, kW, kKeep, kSolo>(I, level, level0, g, G, r0 * kW, rounds,
                                                    rounds * kW, S, P, &s_n);
        }
        if (kSolo && lane == 0) s_new[w] = fresh;
        lds_wait();
        __syncthreads();
        if (kSolo) {
            uint32_t f = 0;
            for (int q = 0; q < kW; ++q) f += s_new[q];
            __syncthreads();  // s_new is free again
            close(level, f);
            if (done >= total) return;
            if (f == 0) {  // impossible for a partial order
                if (tid == 0) atomicOr(&I.sc->err, (uint32_t)kErrInternal);
                return;
            }
        }
    }
}

template <int M, bool kSolo>
__global__ __launch_bounds__(kRankWaves * kWave) void k_ranks(PairInst I) {
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    __shared__ uint32_t s_new[kRankWaves];
    __shared__ uint32_t s_f;
    __shared__ int32_t s_n;
    __shared__ int32_t s_team[2];
    if (I.sc->err) return;
    if constexpr (kSolo) {
        rank_levels<M, kRankWaves, true, true>(I, 0, 1, 0, dyn, s_new, &s_f, &s_n);
    } else {
        rank_team(I, s_team);
        const int32_t g = uniform(s_team[0]), G = uniform(s_team[1]);
        if (G == 0) return;
        if (2 * I.nB <= G * kRankWaves)
            rank_levels<M, kRankWaves, true, false>(I, g, G, 0, dyn, s_new, &s_f, &s_n);
        else
            rank_levels<M, kRankWaves, false, false>(I, g, G, 0, dyn, s_new, &s_f, &s_n);
    }
}

// The levels that the fronts taken off in `phases` phases leave (how many and
// their number of points is on the device).
template <int M>
__global__ __launch_bounds__(kRestWaves * kWave) void k_ranks_rest(PairInst I, int32_t phases) {
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    __shared__ uint32_t s_new[kRestWaves];
    __shared__ uint32_t s_f;
    __shared__ int32_t s_n;
    __shared__ int32_t s_team[2];
    if (I.sc->err) return;
    phases = phase_at(I, phases).taken;
    I = phase_inst(I, phases);
    rank_team(I, s_team);
    const int32_t g = uniform(s_team[0]), G = uniform(s_team[1]);
    if (G == 0) return;
    if (2 * I.nB <= G * kRestWaves)
        rank_levels<M, kRestWaves, true, false>(I, g, G, phases, dyn, s_new, &s_f, &s_n);
    else
        rank_levels<M, kRestWaves, false, false>(I, g, G, phases, dyn, s_new, &s_f, &s_n);
}

// Problems that one work-group holds, a slot a wave.
static bool rank_solo(const PairInst &I, int phases) {
    return phases == 0 && 2 * I.nB <= kRankWaves;
}

// LDS of a rank launch whose waves hold `rounds` slots each.  (Fewer blocks than
// at the start may bring the mask units into LDS.)
static size_t ranks_lds_bytes(const PairInst &I, int phases, int rounds) {
    const int waves = phases > 0 ? kRestWaves : kRankWaves;
    return 4 * (rank_lds_words(I.nBpad, I.M, I.lowK, rounds * waves, rank_solo(I, phases), nullptr,
                               nullptr) +
                (phases > 0 ? kRankIdxWords : 0));
}

void rank_shape(PairInst &I, int max_groups, int started) {
    constexpr size_t kLds = 163840 - 512;  // (the rest is the launches' static part)
    const int phases = pair_phases(I.N, I.M);
    const int waves = phases ? kRestWaves : kRankWaves;
    const int full = (2 * I.nB + waves - 1) / waves;
    int most = max_groups < kRankMaxGroups ? max_groups : kRankMaxGroups;
    if (most < 1) most = 1;
    I.groups = full < most ? full : most;
    I.started = started > 0 ? started : I.groups;
    I.rounds = (2 * I.nB + I.groups * waves - 1) / (I.groups * waves);
    while (I.rounds > 1 && ranks_lds_bytes(I, phases, I.rounds) > kLds) --I.rounds;
}

template <int M>
static hipError_t launch_ranks(const PairInst &I, int phases, hipStream_t s) {
    const dim3 gr((unsigned)I.started);
    const size_t lds = ranks_lds_bytes(I, phases, I.rounds);
    if (phases > 0)
        hipLaunchKernelGGL(k_ranks_rest<M>, gr, dim3(kRestWaves * kWave), lds, s, I, phases);
    else if (rank_solo(I, phases))
        hipLaunchKernelGGL((k_ranks<M, true>), dim3(1), dim3(kRankWaves * kWave), lds, s, I);
    else
        hipLaunchKernelGGL((k_ranks<M, false>), gr, dim3(kRankWaves * kWave), lds, s, I);
    return hipGetLastError();
}

hipError_t run_ranks(const PairInst &I, int phases, hipStream_t s) {
    switch (I.M) {
#define NSGA3_CASE(m) case m: return launch_ranks<m>(I, phases, s);
        NSGA3_CASE(2) NSGA3_CASE(3) NSGA3_CASE(4) NSGA3_CASE(5) NSGA3_CASE(6) NSGA3_CASE(7)
        NSGA3_CASE(8) NSGA3_CASE(9) NSGA3_CASE(10) NSGA3_CASE(11) NSGA3_CASE(12) NSGA3_CASE(13)
        NSGA3_CASE(14) NSGA3_CASE(15) NSGA3_CASE(16)
#undef NSGA3_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace nsga3
