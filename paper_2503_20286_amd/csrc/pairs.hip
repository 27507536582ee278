// Nondominated sorting in a spatial order (see pairs.h): order, block tables
// and boxes, pair probes, ranks.  Dominance is Listing 1 / Eq. (6) on order
// keys (minimisation); degrees are Eq. (7) and the out-degrees beside it, the
// levels Eq. (8)-(9), the last front the end of Sec. IV-A.1.
#include "pairs.h"

#include "kernels.h"
#include "prims.h"
#include "stage_math.h"

namespace nsga3 {

// ---------------------------------------------------------------------------
// order: splitters per objective, cell counts, placement, order inside a cell
// ---------------------------------------------------------------------------
// Sorts one value a thread by a bitonic network.
__device__ __forceinline__ void sort_sample(uint32_t v, uint32_t *s) {
    const int t = (int)threadIdx.x;
    for (int len = 2; len <= kSplitterSample; len <<= 1) {
        for (int d = len >> 1; d > 0; d >>= 1) {
            uint32_t o;
            if (d >= kWave) {  // (the partner is in another wave)
                s[t] = v;
                __syncthreads();
                o = s[t ^ d];
                __syncthreads();
            } else {
                o = (uint32_t)__shfl_xor((int)v, d, kWave);
            }
            const bool low = ((t & len) == 0) == ((t & d) == 0);
            v = low ? (o < v ? o : v) : (o > v ? o : v);
        }
    }
    s[t] = v;
    __syncthreads();
}

// Sampled points: one of each of up to kSplitterSample equal stretches, anywhere in
// it, so that populations with a period are met in all its places.
__device__ __forceinline__ int sample_size(const PairInst &I) {
    return I.N < kSplitterSample ? I.N : kSplitterSample;
}
__device__ __forceinline__ uint32_t sample_point(const PairInst &I, int t) {
    const uint32_t N = (uint32_t)I.N, u = (uint32_t)t;  // (t N < 2^28)
    if (N < (uint32_t)kSplitterSample) return u < N ? u : 0u;
    const uint32_t a = u * N / kSplitterSample, b = (u + 1u) * N / kSplitterSample;
    return a + __umulhi(u * 0x9e3779b1u, b - a);
}

// Hash of a row of keys, 22 bits.
__device__ __forceinline__ uint32_t row_hash(uint32_t h, uint32_t key) {
    h = (h ^ key) * 0x85ebca6bu;
    return h ^ (h >> 15);
}
__device__ __forceinline__ int hash_key(int q, int M) { return M <= 5 ? q : q * M / 5; }
__device__ __forceinline__ uint32_t row_hash_end(uint32_t h) { return (h * 0xc2b2ae35u) >> 10; }

// Quantile splitters of objective k < M from the sample; k == M: the rows that it
// holds kHeavySample times (one point in 64 or more is identical to each), which
// get cells of their own, in which nothing is compared (200k identical rows, M =
// 5: the call 81 ms when each counted its cell, 22.7 by searches in it, 15.6 so, of
// which 15.1 go to the one reference's bucket).
// Only the order of the points depends on either, never a result.
__device__ __forceinline__ void sample_item(const PairInst &I, int k, uint32_t *s, uint32_t *lds) {
    const int M = I.M;
    const int S = sample_size(I);
    const int t = (int)threadIdx.x;
    const float *row = I.objs + (int64_t)sample_point(I, t) * M;
    uint32_t v;
    if (k < M) {
        v = order_key(row[k]);
    } else if (I.N <= kHeavyMinN) {
        if (t == 0) I.heavy[0] = 0u;
        return;
    } else {
        // (five keys tell rows apart well enough, the cells' codes compare them all)
        float f[5];
#pragma unroll
        for (int q = 0; q < 5; ++q)
            if (q < M) f[q] = row[hash_key(q, M)];
        v = 0;
#pragma unroll
        for (int q = 0; q < 5; ++q)
            if (q < M) v = row_hash(v, order_key(f[q]));
        v = row_hash_end(v) << 10 | (uint32_t)t;
        // nothing to sort unless some bucket of hashes holds as many
        s[t] = 0u;
        __syncthreads();
        if (t < S) atomicAdd(&s[v >> 22], 1u);
        lds_wait();
        __syncthreads();
        const uint32_t c = s[t];
        if (!__syncthreads_or(c >= (uint32_t)kHeavySample)) {
            if (t == 0) I.heavy[0] = 0u;
            return;
        }
    }
    sort_sample(t < S ? v : 0xffffffffu, s);  // (one copy of it: the launch waits for its code, too)
    if (k < M) {
        const int n = 1 << I.bits[k];
        if (t < n - 1) I.spl[k * 64 + t] = s[(int)((int64_t)(t + 1) * S / n)];
        return;
    }
    const uint32_t g = s[t] >> 10;
    const bool is = (t == 0 || s[t - 1] >> 10 != g) && t + kHeavySample <= S &&
                    s[t + kHeavySample - 1] >> 10 == g;
    uint32_t n;
    const uint32_t j = block_exclusive_scan(is ? 1u : 0u, lds, &n);  // ascending in the hash
    if (t == 0) I.heavy[0] = n < (uint32_t)kHeavyRows ? n : (uint32_t)kHeavyRows;
    if (is && j < (uint32_t)kHeavyRows) {
        uint32_t *e = I.heavy + 1 + j * (uint32_t)(M + 1);
        row = I.objs + (int64_t)sample_point(I, (int)(s[t] & 1023u)) * M;
        e[0] = g;
        for (int q = 0; q < M; ++q) e[1 + q] = order_key(row[q]);
    }
}

// Splitters (block k < M: objective k), heavy rows (block M), the call's scalars,
// and zeros for the counters.
__global__ __launch_bounds__(kSplitterSample) void k_pair_setup(PairInst I, uint32_t *zero,
                                                                int64_t nzero, int nfill) {
    __shared__ uint32_t s[kSplitterSample];
    __shared__ uint32_t lds[kSplitterSample / kWave + 1];
    if ((int)blockIdx.x <= I.M) {
        sample_item(I, (int)blockIdx.x, s, lds);
        return;
    }
    const int b = (int)blockIdx.x - I.M - 1;
    if (b == 0) {
        init_scalars(I.sc, (int)threadIdx.x);
        if (threadIdx.x < kWBlk)
            I.mask[(size_t)I.allUnit * kWBlk + threadIdx.x] = make_uint4(~0u, ~0u, ~0u, ~0u);
    }
    const int64_t t = (int64_t)b * kSplitterSample + threadIdx.x;
    for (int64_t q = t; q < nzero; q += (int64_t)nfill * kSplitterSample) zero[q] = 0u;
}

// Cell of every point, its arrival position in the cell, ideal point, finiteness.
__global__ __launch_bounds__(256) void k_cell_code(PairInst I) {
    __shared__ uint32_t spl[16 * 64];
    __shared__ uint32_t smin[16];
    const int M = I.M;
    for (int q = threadIdx.x; q < M * 64; q += 256)
        spl[q] = (q & 63) < (1 << I.bits[q >> 6]) - 1 ? I.spl[q] : 0xffffffffu;
    if (threadIdx.x < 16) smin[threadIdx.x] = 0xffffffffu;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool in = i < I.N;
    bool bad = false;
    uint32_t code = 0;
    uint32_t bk[16];
    const int nh = (int)I.heavy[0];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        if (k < M) {
            const float f = in ? I.objs[i * M + k] : 0.0f;
            bad |= !__builtin_isfinite(f);
            const uint32_t key = order_key(f);
            const uint32_t v = wave_min(in ? key : 0xffffffffu);
            if (lane_id() == 0) atomicMin(&smin[k], v);
            const int nb = I.bits[k];
            uint32_t c = 0;  // splitters <= key
            for (int st = nb - 1; st >= 0; --st)
                if (spl[k * 64 + c + (1u << st) - 1u] <= key) c += 1u << st;
            bk[k] = c;
        } else {
            bk[k] = 0;
        }
    }
    int top = 0;
    for (int k = 0; k < M; ++k) top = max(top, (int)I.bits[k]);
    for (int pl = top - 1; pl >= 0; --pl)
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (k < M && pl < (int)I.bits[k]) code = (code << 1) | ((bk[k] >> pl) & 1u);
    if (ballot(bad) && lane_id() == 0) atomicOr(&I.sc->err, (uint32_t)kErrNonfiniteObj);
    if (nh > 0 && in) {
        uint32_t hash = 0;
        for (int q = 0; q < 5 && q < M; ++q)
            hash = row_hash(hash, order_key(I.objs[i * M + hash_key(q, M)]));
        hash = row_hash_end(hash);
        int j = 0;  // heavy rows of smaller hash
        for (int s = nh; s > 0;) {
            const int q = s >> 1;
            const bool go = I.heavy[1 + (j + q) * (M + 1)] < hash;
            j = go ? j + q + 1 : j;
            s = go ? s - q - 1 : q;
        }
        if (j < nh) {
            const uint32_t *e = I.heavy + 1 + j * (M + 1);
            bool eq = e[0] == hash;
            for (int k = 0; k < M && eq; ++k) eq = e[1 + k] == order_key(I.objs[i * M + k]);
            if (eq) code = (uint32_t)(pair_heavy_cell(I.T) + j);
        }
    }
    // points of a wave that share a cell take one atomic, where they are many
    // (heavy rows, wide cells)
    uint32_t slot = 0;
    uint64_t act = ballot(in), ask = act;
    const uint64_t heavy = nh > 0 ? ballot(in && code >= (uint32_t)pair_heavy_cell(I.T)) : 0ull;
    for (int q = 0; q < 4 && ask; ++q) {
        const int l = __builtin_ctzll(ask & heavy ? ask & heavy : ask);
        const uint32_t c0 = (uint32_t)__builtin_amdgcn_readlane((int)code, l);
        const uint64_t same = ballot(((act >> lane_id()) & 1) != 0 && code == c0);
        ask &= ~same;
        if (__popcll(same) < 8) continue;
        uint32_t n = 0;
        if ((int)lane_id() == l) n = atomicAdd(&I.cell[c0], (uint32_t)__popcll(same));
        n = (uint32_t)__builtin_amdgcn_readlane((int)n, l) + lanes_below(same);
        if ((same >> lane_id()) & 1) slot = n;
        act &= ~same;
    }
    if ((act >> lane_id()) & 1) slot = atomicAdd(&I.cell[code], 1u);
    if (in) {
        I.code[i] = code;
        I.slot[i] = slot;
    }
    __syncthreads();
    if ((int)threadIdx.x < M) atomicMin(&I.sc->min_key[threadIdx.x], smin[threadIdx.x]);
}

// Block 0: exclusive scan of the cell counts.  Other blocks: the unit
// references.
__global__ __launch_bounds__(1024) void k_cell_scan(PairInst I, RefArgs R) {
    __shared__ uint32_t lds[17];
    if (blockIdx.x > 0) {
        reference_item(R, I.M, (int)(blockIdx.x - 1) * 1024 + (int)threadIdx.x, I.sc);
        return;
    }
    // a thread's up to 68 consecutive counts stay in registers between the sum
    // and the starts (65536 cells: 24 us when they were read one by one, twice)
    const int n = pair_cells(I.T);
    constexpr int kVec = ((1 << kCellMaxBits) + kHeavyRows + 4095) / 4096;
    const int per = (n + 4095) / 4096 * 4;
    const int s0 = (int)threadIdx.x * per;
    uint32_t *c = I.cell + s0;
    uint32_t v[4 * kVec];
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        uint4 x = make_uint4(0, 0, 0, 0);
        if (4 * q < per && s0 + 4 * q < n) x = *reinterpret_cast<const uint4 *>(c + 4 * q);
        v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        sum += x.x + x.y + x.z + x.w;
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(sum, lds, &tot);
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        uint4 x;
        x.x = run;
        x.y = x.x + v[4 * q];
        x.z = x.y + v[4 * q + 1];
        x.w = x.z + v[4 * q + 2];
        run = x.w + v[4 * q + 3];
        if (4 * q < per && s0 + 4 * q < n) *reinterpret_cast<uint4 *>(c + 4 * q) = x;
    }
    if (threadIdx.x == 0) I.cell[n] = tot;
}

// Records (keys, point index) into cell order.
__global__ __launch_bounds__(256) void k_cell_place(PairInst I) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= I.N) return;
    const int M = I.M, MP = rec_stride(M);
    const uint32_t p = I.cell[I.code[i]] + I.slot[i];
    uint4 *dst = reinterpret_cast<uint4 *>(I.trec + (size_t)p * MP);
    for (int q = 0; q < MP / 4; ++q) {
        uint32_t v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = 4 * q + t;
            v[t] = k < M ? order_key(I.objs[i * M + k]) : (k == M ? (uint32_t)i : 0u);
        }
        dst[q] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

// Final position: inside its cell a point comes after every lexicographically
// smaller row and every identical row of smaller index, so identical rows end
// up adjacent (they share a cell).  A point counts its cell alone where that is
// small; the splitters cut each objective by itself, so identical rows and
// objectives that move together may put any share of the points into one cell.
constexpr int kCellOwn = 256;     // positions of a work-group
// Points of a cell that a point counts alone.  (64 / 128 / 256, all cells: rows
// that move together in part, N = 34k, M = 16, 91 / 120 / 152 us, N = 20k, M = 5, 69 / 52 / 48;
// a front of N = 200k, M = 5, whose cells hold up to 87, 71 / 34 / 34.)
constexpr uint32_t kCellWide = 128;

// Record, point index and run of identical rows [run, end) of position at.
template <int M>
__device__ __forceinline__ void put_row(const PairInst &I, const uint32_t (&x)[M], uint32_t i,
                                        uint32_t at, uint32_t run, uint32_t end) {
    constexpr int MP = rec_stride(M);
    uint32_t v[MP];
#pragma unroll
    for (int k = 0; k < MP; ++k) v[k] = k < M ? x[k < M ? k : 0] : (k == M ? at : 0u);
    uint4 *dst = reinterpret_cast<uint4 *>(I.recs + (size_t)at * MP);
#pragma unroll
    for (int q = 0; q < MP / 4; ++q)
        dst[q] = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    I.sval[at] = i;
    I.runs[at] = (int32_t)run;
    I.rune[at] = (int32_t)end;
}

// A wide cell [c0, c1), of which the work-group has the points at positions
// [a, b): they are put in order in LDS, and every point of the cell is looked up
// among them; the numbers of points that fall between them give each one's
// place.  The cell costs a work-group its size / 256 times a search of 8 steps
// instead of its size.  First keys decide nearly always; the others are read only
// where two are equal.  (Rows near one line, N = 200k, M = 5, 27k points in a cell:
// the call 19.4 ms when each point counted its cell, 13.9 so.)
template <int M>
struct WideCell {
    uint32_t key[M][kCellOwn];
    uint32_t idx[kCellOwn];
    uint32_t le[kCellOwn + 1], lt[kCellOwn + 1], at[kCellOwn + 1];
    uint32_t scan[kCellOwn / kWave + 1];
};

template <int M>
__device__ __forceinline__ void wide_cell(const PairInst &I, WideCell<M> &W, uint32_t c0, uint32_t c1,
                                          uint32_t a, uint32_t b) {
    constexpr int MP = rec_stride(M);
    const int t = (int)threadIdx.x;
    const int n = (int)(b - a);
    {
        // (places past the last point: after every row)
        const uint32_t *r = I.trec + (size_t)(t < n ? a + (uint32_t)t : a) * MP;
#pragma unroll 1
        for (int k = 0; k < M; ++k) W.key[k][t] = t < n ? r[k] : 0xffffffffu;
        W.idx[t] = t < n ? r[M] : 0xffffffffu;
    }
    // a bitonic network moves first keys and places
    uint32_t a0 = W.key[0][t], p = (uint32_t)t;
#pragma unroll 1
    for (int len = 2; len <= kCellOwn; len <<= 1) {
#pragma unroll 1
        for (int d = len >> 1; d > 0; d >>= 1) {
            __syncthreads();
            W.le[t] = a0;
            W.lt[t] = p;
            __syncthreads();
            const uint32_t b0 = W.le[t ^ d], r = W.lt[t ^ d];
            int o = a0 < b0 ? -1 : (a0 > b0 ? 1 : 0);
            if (a0 == 0xffffffffu && o == 0) o = p < r ? -1 : 1;  // (past the last point)
            if (ballot(o == 0)) {
#pragma unroll 1
                for (int k = 1; k < M && ballot(o == 0); ++k) {
                    const uint32_t v = W.key[k][p], w = W.key[k][r];
                    o = o != 0 ? o : (v < w ? -1 : (v > w ? 1 : 0));
                }
                const uint32_t v = W.idx[p], w = W.idx[r];
                o = o != 0 ? o : (v < w ? -1 : 1);
            }
            if ((o < 0) != (((t & len) == 0) == ((t & d) == 0))) {
                a0 = b0;
                p = r;
            }
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k <= M; ++k) {  // (the rows after them)
        uint32_t *row = k < M ? W.key[k < M ? k : 0] : W.idx;
        const uint32_t v = row[p];
        __syncthreads();
        row[t] = v;
        lds_wait();
        __syncthreads();
    }
    for (int q = t; q <= kCellOwn; q += kCellOwn) W.le[q] = W.lt[q] = W.at[q] = 0u;
    lds_wait();
    __syncthreads();
    // four of a thread side by side: by the first key alone, where no other row here
    // has it
    constexpr int kAhead = 4;
#pragma unroll 1
    for (uint32_t q0 = c0; q0 < c1; q0 += kAhead * kCellOwn) {
        uint32_t y[kAhead];
        int at[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            y[u] = I.trec[(size_t)min(q0 + (uint32_t)(u * kCellOwn + t), c1 - 1u) * MP];
            at[u] = 0;
        }
#pragma unroll
        for (int s = kCellOwn / 2; s > 0; s >>= 1)
#pragma unroll
            for (int u = 0; u < kAhead; ++u) at[u] += W.key[0][at[u] + s - 1] < y[u] ? s : 0;
        bool tie[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t v = W.key[0][at[u]];
            at[u] += v < y[u] ? 1 : 0;   // (the last place)
            const uint32_t q = q0 + (uint32_t)(u * kCellOwn + t);
            const bool same = v == y[u];
            // (a row of the work-group's own, the only one of its first key)
            const bool own = same && q >= a && q < b &&
                             (at[u] + 1 >= n || W.key[0][at[u] + 1] != y[u]);
            tie[u] = same && !own && q < c1;
            if (q < c1 && !tie[u]) {
                atomicAdd(&W.le[at[u]], 1u);
                atomicAdd(&W.lt[at[u] + (own ? 1 : 0)], 1u);
                atomicAdd(&W.at[at[u] + (own ? 1 : 0)], 1u);
            }
        }
#pragma unroll 1
        for (int u = 0; u < kAhead; ++u) {
            const bool on = u == 0 ? tie[0] : u == 1 ? tie[1] : u == 2 ? tie[2] : tie[3];
            if (!on) continue;
            const uint32_t q = q0 + (uint32_t)(u * kCellOwn + t);
            const uint32_t *row = I.trec + (size_t)q * MP;
            const uint4 f = *reinterpret_cast<const uint4 *>(row);
            const uint32_t g[4] = {f.x, f.y, f.z, f.w}, y0 = f.x;
            // points here before the row (first search), and not after it (second)
            int pos = 0, lo = 0;
#pragma unroll 1
            for (int up = 0; up < 2; ++up) {
                for (int s = n - pos; s > 0;) {
                    const int h = s >> 1;
                    const uint32_t v0 = W.key[0][pos + h];
                    int o = y0 < v0 ? -1 : (y0 > v0 ? 1 : 0);
#pragma unroll
                    for (int k = 1; k < 4 && k < M; ++k) {
                        const uint32_t v = W.key[k][pos + h];
                        o = o != 0 ? o : (g[k] < v ? -1 : (g[k] > v ? 1 : 0));
                    }
#pragma unroll 1
                    for (int k = 4; k < M && ballot(o == 0); ++k) {
                        const uint32_t x = row[k], v = W.key[k][pos + h];
                        o = o != 0 ? o : (x < v ? -1 : (x > v ? 1 : 0));
                    }
                    const bool go = o > 0 || (up != 0 && o == 0);
                    pos = go ? pos + h + 1 : pos;
                    s = go ? s - h - 1 : h;
                }
                if (up == 0) lo = pos;
                if (pos >= n || W.key[0][pos] != y0) break;
            }
            int e = lo;       // and those of its row up to its own index
            if (pos > lo) {
                const uint32_t yi = row[M];
                for (int s = pos - lo; s > 0;) {
                    const int h = s >> 1;
                    const bool go = W.idx[e + h] <= yi;
                    e = go ? e + h + 1 : e;
                    s = go ? s - h - 1 : h;
                }
            }
            atomicAdd(&W.le[lo], 1u);
            atomicAdd(&W.lt[pos], 1u);
            atomicAdd(&W.at[e], 1u);
        }
    }
    lds_wait();
    __syncthreads();
    // point s comes after every y that falls at s or before
    uint32_t tot, sum[3];
#pragma unroll 1
    for (int h = 0; h < 3; ++h) {
        const uint32_t v = (h == 0 ? W.le : h == 1 ? W.lt : W.at)[t];
        const uint32_t s = v + block_exclusive_scan(v, W.scan, &tot);
        sum[0] = h == 0 ? s : sum[0];
        sum[1] = h == 1 ? s : sum[1];
        sum[2] = h == 2 ? s : sum[2];
        __syncthreads();
    }
    if (t < n) {
        const uint32_t at = c0 + sum[2];
        uint32_t *dst = I.recs + (size_t)at * MP;
#pragma unroll 1
        for (int k = 0; k < MP; ++k) dst[k] = k < M ? W.key[k < M ? k : 0][t] : (k == M ? at : 0u);
        I.sval[at] = W.idx[t];
        I.runs[at] = (int32_t)(c0 + sum[1]);
        I.rune[at] = (int32_t)(c0 + sum[0]);
    }
    lds_wait();
    __syncthreads();
}

template <int M>
__global__ __launch_bounds__(kCellOwn) void k_cell_sort(PairInst I) {
    constexpr int MP = rec_stride(M);
    __shared__ WideCell<M> W;
    __shared__ uint32_t s_from;
    const uint32_t p0 = blockIdx.x * (uint32_t)kCellOwn, p = p0 + threadIdx.x, N = (uint32_t)I.N;
    uint32_t c0 = 0, c1 = 0;
    if (p < N) {
        uint32_t x[M];
#pragma unroll
        for (int k = 0; k < M; ++k) x[k] = I.trec[(size_t)p * MP + k];
        const uint32_t i = I.trec[(size_t)p * MP + M];
        const uint32_t c = I.code[i];
        c0 = I.cell[c];
        c1 = I.cell[c + 1];
        if (c >= (uint32_t)pair_heavy_cell(I.T)) {  // identical rows, in any order
            put_row<M>(I, x, i, p, c0, c1);
            c1 = c0;
        } else if (c1 - c0 <= kCellWide) {
            uint32_t less = 0, same = 0, before = 0;
#pragma unroll 4
            for (uint32_t q = c0; q < c1; ++q) {
                const uint32_t *r = I.trec + (size_t)q * MP;
                bool lt = false, eq = true;
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const uint32_t y = r[k];
                    lt = lt || (eq && y < x[k]);
                    eq = eq && y == x[k];
                }
                less += lt ? 1u : 0u;
                same += eq ? 1u : 0u;
                before += (eq && r[M] < i) ? 1u : 0u;
            }
            const uint32_t run = c0 + less;
            put_row<M>(I, x, i, run + before, run, run + same);
        }
    }
    const bool wide = c1 - c0 > kCellWide;
    if (!__syncthreads_or(wide)) return;
    // the wide cells of the work-group's positions, in order (its first points here tell)
    for (uint32_t from = p0;;) {
        if (threadIdx.x == 0) s_from = 0xffffffffu;
        __syncthreads();
        if (wide && p >= from) atomicMin(&s_from, p);
        lds_wait();
        __syncthreads();
        const uint32_t a = s_from;
        if (a == 0xffffffffu) return;
        __syncthreads();
        __shared__ uint32_t s_c[2];
        if (p == a) { s_c[0] = c0; s_c[1] = c1; }
        lds_wait();
        __syncthreads();
        const uint32_t d0 = s_c[0], d1 = s_c[1];
        const uint32_t end = min(p0 + (uint32_t)kCellOwn, N), b = min(d1, end);
        wide_cell<M>(I, W, d0, d1, a, b);
        from = b;
    }
}

// Small problems: the whole order by one work-group of a thread a point.  A
// handful of blocks needs no cells: the rows are put in lexicographic order by
// counting.  Four launches less, and the splitters (N = 200, M = 3: 94 us a
// call with them).  One CU makes all N x N x M compares, so the line is at N x M:
// by one work-group / by cells M = 2, N = 512 148 / 149 us, 640 194 / 176; M = 5, N = 128
// 93 / 98, 256 111 / 104, 1024 334 / 124; M = 16, N = 64 145 / 144, 1024 878 / 175.
constexpr int kOrderOne = 1024;
constexpr int kOrderOneKeys = 1024;
constexpr int kOrderOneRefs = 4096;   // (it also scales the references, and clears their counters)

template <int M>
__global__ __launch_bounds__(kOrderOne) void k_order_one(PairInst I, RefArgs R, uint32_t *zero,
                                                         int64_t nzero) {
    __shared__ uint32_t row[kOrderOneKeys];
    __shared__ uint32_t smin[M];
    const int t = (int)threadIdx.x;
    init_scalars(I.sc, t);
    if (t < kWBlk) I.mask[(size_t)I.allUnit * kWBlk + t] = make_uint4(~0u, ~0u, ~0u, ~0u);
    for (int64_t q = t; q < nzero; q += kOrderOne) zero[q] = 0u;
    const int N = I.N;
    const bool in = t < N;
    bool bad = false;
    uint32_t x[M];
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const float f = in ? I.objs[(int64_t)t * M + k] : 0.0f;
        bad |= !__builtin_isfinite(f);
        x[k] = order_key(f);
        if (in) row[t * M + k] = x[k];
    }
    if (t < M) smin[t] = 0xffffffffu;
    __syncthreads();  // (the scalars, too)
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const uint32_t v = wave_min(in ? x[k] : 0xffffffffu);
        if (lane_id() == 0) atomicMin(&smin[k], v);
    }
    if (ballot(bad) && lane_id() == 0) atomicOr(&I.sc->err, (uint32_t)kErrNonfiniteObj);
    for (int j = t; j < R.Hpad; j += kOrderOne) reference_item(R, M, j, I.sc);
    uint32_t less = 0, same = 0, before = 0;
    if (in) {
        for (int q = 0; q < N; ++q) {
            bool lt = false, eq = true;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const uint32_t y = row[q * M + k];
                lt = lt || (eq && y < x[k]);
                eq = eq && y == x[k];
            }
            less += lt ? 1u : 0u;
            same += eq ? 1u : 0u;
            before += (eq && q < t) ? 1u : 0u;
        }
        put_row<M>(I, x, (uint32_t)t, less + before, less, less + same);
    }
    __syncthreads();
    if (t < M) I.sc->min_key[t] = smin[t];
}

// ---------------------------------------------------------------------------
// tables and boxes: one block of 128 points per work-group, a wave per objective
// ---------------------------------------------------------------------------
// kStep: after `step` fronts were taken off (0 without).
template <int M, bool kStep>
__global__ __launch_bounds__(M * kWave) void k_pair_build(PairInst I, int32_t step) {
    __shared__ int32_t inv[M][kWBlk];
    if (I.sc->err) return;
    if constexpr (kStep) {
        if (phase_at(I, step).taken != step) return;
        I = phase_inst(I, step);
    }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t b = (int32_t)blockIdx.x;
    if (b >= I.nB) return;
    uint32_t *T = I.tabs + (size_t)b * wblk_stride(M);
    build_wide_at<M>(I.recs, I.N, T, b, inv[w], w, M);
    // the block's box: entries past the last point repeat it
    constexpr int MP = rec_stride(M);
    const int l = (int)lane_id();
    const int32_t e0 = b * kWBlk + l, e1 = e0 + kWave;
    const uint32_t x0 = I.recs[(size_t)min(e0, I.N - 1) * MP + w];
    const uint32_t x1 = I.recs[(size_t)min(e1, I.N - 1) * MP + w];
    const uint32_t l0 = wave_extreme<false>(x0), l1 = wave_extreme<false>(x1);
    const uint32_t hi = wave_extreme<true>(x0 > x1 ? x0 : x1);
    if (l == 0) {
        I.box[(size_t)w * I.nBpad + b] = l0 < l1 ? l0 : l1;
        I.box[(size_t)(M + w) * I.nBpad + b] = hi;
        I.low[(size_t)(2 * b) * 16 + w] = l0;
        I.low[(size_t)(2 * b + 1) * 16 + w] = l1;
    }
}

// ---------------------------------------------------------------------------
// pairs: one wave holds a tile of 128 points (two per lane, a block of the
// order); a work-group's tiles meet the tables of a range of blocks.
// ---------------------------------------------------------------------------
// Mask words of objective k of table T for two keys: members with key <= x
// (kLe) or < x.
template <bool kLe>
__device__ __forceinline__ void probe2(uint32_t base, int k, uint32_t xa, uint32_t xb,
                                       uint32_t (&ma)[4], uint32_t (&mb)[4]) {
    const uint32_t o = base + 4u * (uint32_t)wblk_obj_off(k);
    auto in = [](uint32_t v, uint32_t x) { return kLe ? v <= x : v < x; };
    uint32_t a, b;
    {
        const uint32_t v = lds_ld(o + 4u * (uint32_t)(kWRegion + 31));  // key 63
        a = o + (in(v, xa) ? 4u * 2u * kWRegion : 0u);
        b = o + (in(v, xb) ? 4u * 2u * kWRegion : 0u);
    }
    {
        const uint32_t va = lds_ld(a + 4u * 31u), vb = lds_ld(b + 4u * 31u);
        a += in(va, xa) ? 4u * kWRegion : 0u;
        b += in(vb, xb) ? 4u * kWRegion : 0u;
    }
#pragma unroll
    for (int step = 16; step >= 1; step >>= 1) {
        const uint32_t va = lds_ld(a + 4u * (uint32_t)(step - 1));
        const uint32_t vb = lds_ld(b + 4u * (uint32_t)(step - 1));
        a += in(va, xa) ? 4u * step : 0u;
        b += in(vb, xb) ? 4u * step : 0u;
    }
    {
        const uint32_t va = lds_ld(a), vb = lds_ld(b);
        a += in(va, xa) ? 4u : 0u;
        b += in(vb, xb) ? 4u : 0u;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        ma[q] = lds_ld(a + 4u * (uint32_t)(32 + 33 * q));
        mb[q] = lds_ld(b + 4u * (uint32_t)(32 + 33 * q));
    }
}

// 64 x 64 bit transpose across the wave: lane r holds row r (lo: columns 0-31,
// hi: columns 32-63); afterwards lane c holds column c.  Blocks of 32 and 16
// rows trade places by lane-group swaps, smaller ones by lane permutes with a
// rotate and a bit select.
struct Transpose64 {
    uint32_t sel16, sel8, k4, k2, k1, a4, a2, a1;
    __device__ __forceinline__ Transpose64() {
        const uint32_t l = lane_id();
        // v_perm bytes: 0-3 of the second operand, 4-7 of the first
        sel16 = (l & 16u) ? 0x07060302u : 0x05040100u;
        sel8 = (l & 8u) ? 0x07030501u : 0x02060004u;
        k4 = (l & 4u) ? 0xf0f0f0f0u : 0x0f0f0f0fu;
        k2 = (l & 2u) ? 0xccccccccu : 0x33333333u;
        k1 = (l & 1u) ? 0xaaaaaaaau : 0x55555555u;
        a4 = (l & 4u) ? 4u : 28u;
        a2 = (l & 2u) ? 2u : 30u;
        a1 = (l & 1u) ? 1u : 31u;
    }
    template <int kCtrl>
    static __device__ __forceinline__ uint32_t dpp(uint32_t x) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, kCtrl, 0xf, 0xf, false);
    }
    __device__ __forceinline__ uint32_t word(uint32_t x) const {
        {
            const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
            x = __builtin_amdgcn_perm(r[1], r[0], sel16);
        }
        x = __builtin_amdgcn_perm(x, dpp<0x128>(x), sel8);          // row_ror:8
        uint32_t y = dpp<0x1b>(dpp<0x141>(x));                      // lane ^ 4: half mirror, quad 3210
        x = (x & k4) | (__builtin_amdgcn_alignbit(y, y, a4) & ~k4);
        y = dpp<0x4e>(x);                                           // lane ^ 2
        x = (x & k2) | (__builtin_amdgcn_alignbit(y, y, a2) & ~k2);
        y = dpp<0xb1>(x);                                           // lane ^ 1
        x = (x & k1) | (__builtin_amdgcn_alignbit(y, y, a1) & ~k1);
        return x;
    }
    __device__ __forceinline__ void run(uint32_t &lo, uint32_t &hi) const {
        const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        lo = word(r[0]);
        hi = word(r[1]);
    }
};

// nv vectors of a table between memory and LDS through V registers a thread.
typedef uint32_t vec4 __attribute__((ext_vector_type(4)));
template <int V, int nv>
__device__ __forceinline__ void load_vec(vec4 (&r)[V], const uint32_t *src) {
    const vec4 *s4 = reinterpret_cast<const vec4 *>(src);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int q = v * kPairWaves * kWave + (int)threadIdx.x;
        r[v] = s4[q < nv ? q : nv - 1];
    }
}
template <int V, int nv>
__device__ __forceinline__ void store_vec(uint32_t *dst, const vec4 (&r)[V]) {
    vec4 *d4 = reinterpret_cast<vec4 *>(dst);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int q = v * kPairWaves * kWave + (int)threadIdx.x;
        if (q < nv) d4[q] = r[v];
    }
}

// Dominators of the points of tile group tg in up to 64 blocks: a lane holds a
// block `blk` of the set `group` and the objectives `need` in which its box
// does not lie below the wave's tile; the tile meets the blocks `mine`.
// Degrees, and (kMask) the masks of the pairs that have any.  kOut:
// out-degrees too (the masks transposed: each lane counts the points a member
// dominates), summed in LDS over the work-group's tiles.
template <int M, bool kOut, bool kMask>
__device__ __forceinline__ void pair_blocks(const PairInst &I, int32_t tg, int32_t blk,
                                            uint32_t need, uint64_t group, uint64_t mine, int pool,
                                            uint32_t *lt, uint32_t *oc) {
    constexpr int MP = rec_stride(M);
    constexpr int TS = wblk_stride(M);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = (int)lane_id();
    const int32_t N = I.N, nBp = I.nBpad;
    const int32_t tile = tg * kPairWaves + w;
    uint64_t stored = 0;
    uint32_t x0[M], x1[M];
    int32_t r0 = 0, r1 = 0, e0 = 0, e1 = 0;
    const int32_t q0 = tile * kWBlk + lane, q1 = q0 + kWave;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        x0[k] = q0 < N ? I.recs[(size_t)q0 * MP + k] : 0u;  // dominated by nothing
        x1[k] = q1 < N ? I.recs[(size_t)q1 * MP + k] : 0u;
    }
    if (q0 < N) { r0 = I.runs[q0]; e0 = I.rune[q0]; }
    if (q1 < N) { r1 = I.runs[q1]; e1 = I.rune[q1]; }
    const Transpose64 tr;
    const uint32_t base = lds_addr(lt);
    pool = (pool + w) & (int)I.poolMask;
    int32_t c0 = 0, c1 = 0;
    int32_t prev = -1;
    uint64_t g = group;
    // a table goes to LDS through registers, so that the next one is on its way
    // while this one is probed
    constexpr int kVec = (TS / 4 + kPairWaves * kWave - 1) / (kPairWaves * kWave);
    vec4 ahead[kVec];
    int32_t nxt = __builtin_amdgcn_readlane(blk, __builtin_ctzll(g));
    load_vec<kVec, TS / 4>(ahead, I.tabs + (size_t)nxt * TS);
    if (kOut && threadIdx.x < kWBlk) oc[threadIdx.x] = 0u;
    while (true) {
        const int ai = g ? __builtin_ctzll(g) : -1;
        if constexpr (kOut) lds_wait();
        __syncthreads();  // every wave is done with the previous table
        if (kOut && prev >= 0 && threadIdx.x < kWBlk) {
            const uint32_t v = oc[threadIdx.x];
            if (v) {
                atomicAdd(&I.dout[prev * kWBlk + (int32_t)threadIdx.x], (int32_t)v);
                oc[threadIdx.x] = 0u;
            }
        }
        if (ai < 0) break;
        g &= g - 1;
        const int32_t a = nxt;
        prev = a;
        store_vec<kVec, TS / 4>(lt, ahead);
        __syncthreads();
        // the next table (the last one again at the end) is in flight during the probe
        nxt = __builtin_amdgcn_readlane(blk, g ? __builtin_ctzll(g) : ai);
        load_vec<kVec, TS / 4>(ahead, I.tabs + (size_t)nxt * TS);
        if (!((mine >> ai) & 1)) continue;
        const uint32_t nd = (uint32_t)__builtin_amdgcn_readlane((int)need, ai);
        uint32_t ma[4], mb[4];
        low_bits128(q0 < N ? lt[2] : 0u, ma);
        low_bits128(q1 < N ? lt[2] : 0u, mb);
        bool alive = true;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            if (alive && ((nd >> k) & 1u)) {
                uint32_t pa[4], pb[4];
                probe2<true>(base, k, x0[k], x1[k], pa, pb);
                uint32_t any = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    ma[q] &= pa[q];
                    mb[q] &= pb[q];
                    any |= ma[q] | mb[q];
                }
                alive = ballot(any != 0u) != 0ull;
            }
        }
        if (!alive) continue;
        // rows identical to a point do not dominate it
        const int32_t ab = a * kWBlk;
        bool all = nd == 0u;
        if (ballot((r0 < ab + kWBlk && e0 > ab) || (r1 < ab + kWBlk && e1 > ab))) {
            all = false;
            uint32_t ra[4], rb[4];
            range_bits128(r0 - ab, e0 - ab, ra);
            range_bits128(r1 - ab, e1 - ab, rb);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ma[q] &= ~ra[q];
                mb[q] &= ~rb[q];
            }
        }
        const uint32_t n0 = __popc(ma[0]) + __popc(ma[1]) + __popc(ma[2]) + __popc(ma[3]);
        const uint32_t n1 = __popc(mb[0]) + __popc(mb[1]) + __popc(mb[2]) + __popc(mb[3]);
        if (!ballot((n0 | n1) != 0u)) continue;
        c0 += (int32_t)n0;
        c1 += (int32_t)n1;
        if constexpr (kMask) {
            stored |= 1ull << ai;
            uint32_t at = I.allUnit;  // every member dominates every point
            if (!all) {
                unsigned long long got = 0;
                if (lane == 0)
                    got = atomicAdd((unsigned long long *)&I.sync->pool[pool].v, 1ull);
                const uint32_t unit = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)got);
                at = kUnitNone;
                if (unit < I.poolUnits) {
                    at = (uint32_t)pool * I.poolUnits + unit;
                    uint4 *d = I.mask + (size_t)at * kWBlk;
                    d[lane] = make_uint4(ma[0], ma[1], ma[2], ma[3]);
                    d[kWave + lane] = make_uint4(mb[0], mb[1], mb[2], mb[3]);
                }
            }
            if (lane == 0) I.idx[(size_t)tile * nBp + a] = at;
        }
        if constexpr (kOut) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                tr.run(ma[2 * h], ma[2 * h + 1]);
                tr.run(mb[2 * h], mb[2 * h + 1]);
                const uint32_t n = __popc(ma[2 * h]) + __popc(ma[2 * h + 1]) + __popc(mb[2 * h]) +
                                   __popc(mb[2 * h + 1]);
                if (n) __hip_atomic_fetch_add(oc + h * kWave + lane, n, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    if (c0) atomicAdd(&I.din[q0], c0);
    if (c1) atomicAdd(&I.din[q1], c1);
    if (kMask && ((stored >> lane) & 1))
        atomicOr((unsigned long long *)&I.nz[(size_t)tile * (nBp / 64) + (blk >> 6)],
                 1ull << (blk & 63));
}

// The same for blocks [a0, a0 + na), na <= 64.
template <int M, bool kOut, bool kMask>
__device__ __forceinline__ void pair_item(const PairInst &I, int32_t tg, int32_t a0, int32_t na,
                                          uint32_t *lt, uint32_t *oc) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = (int)lane_id();
    const int32_t nB = I.nB, nBp = I.nBpad;
    const int32_t tile = tg * kPairWaves + w;
    // the lane's block of the range against the tile's box and the work-group's
    uint32_t need = 0;
    const bool la = lane < na;
    const int32_t a = a0 + (la ? lane : 0);
    bool okm = la && tile < nB, okg = la;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const uint32_t alo = I.box[(size_t)k * nBp + a], ahi = I.box[(size_t)(M + k) * nBp + a];
        uint32_t ghi = 0u;
#pragma unroll
        for (int u = 0; u < kPairWaves; ++u) {
            const int32_t tt = min(tg * kPairWaves + u, nB - 1);
            const uint32_t h = I.box[(size_t)(M + k) * nBp + tt];
            ghi = h > ghi ? h : ghi;
        }
        const int32_t tt = min(tile, nB - 1);
        okm = okm && alo <= I.box[(size_t)(M + k) * nBp + tt];
        okg = okg && alo <= ghi;
        need |= ahi > I.box[(size_t)k * nBp + tt] ? 1u << k : 0u;
    }
    const uint64_t mine = ballot(okm), group = ballot(okg);
    if (group)
        pair_blocks<M, kOut, kMask>(I, tg, a, need, group, mine,
                                    5 * tg + a0, lt, oc);
}

// Small problems: a work-group takes a group of kPairWaves tiles against a range
// of G blocks (a power of two), as many as fill the chip.
__host__ __device__ inline int32_t pair_range(int32_t nB) {
    const int32_t tgs = (nB + kPairWaves - 1) / kPairWaves;
    int32_t G = 16;
    while (G > 1 && (int64_t)tgs * ((nB + G - 1) / G) < 2048) G >>= 1;
    return G;
}

template <int M, bool kOut>
__global__ __launch_bounds__(kPairWaves * kWave) void k_pairs(PairInst I, int32_t G) {
    __shared__ __attribute__((aligned(16))) uint32_t lt[wblk_stride(M)];
    __shared__ uint32_t oc[kOut ? kWBlk : 1];
    if (I.sc->err) return;
    const int32_t a0 = (int32_t)blockIdx.y * G;
    pair_item<M, kOut, true>(I, (int32_t)blockIdx.x, a0, min(G, I.nB - a0), lt, oc);
}

// Larger ones: the tile groups' surviving blocks are listed first, kListItem to
// an item; work-groups then take items from a counter.  (Over ranges most of
// 40,000 work-groups found 2 blocks or none, and the tiles at the far corner
// of objective space all 16.)
template <int M>
__global__ __launch_bounds__(256) void k_pair_list(PairInst I, int32_t step) {
    __shared__ uint4 ent[kPairsMaxN / kWBlk];
    __shared__ uint32_t lo[kPairWaves][16], hi[kPairWaves][16];
    __shared__ int32_t s_n, s_base;
    if (I.sc->err) return;
    if (step > 0) {
        if (phase_at(I, step).taken != step) return;
        I = phase_inst(I, step);
    }
    const int32_t nB = I.nB, nBp = I.nBpad;
    const int32_t tg = (int32_t)blockIdx.x;
    if (tg * kPairWaves >= nB) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = (int)lane_id();
    if (threadIdx.x == 0) s_n = 0;
    if (threadIdx.x < kPairWaves * 16) {
        const int u = (int)threadIdx.x / 16, k = (int)threadIdx.x % 16;
        const int32_t tt = tg * kPairWaves + u;
        const bool in = tt < nB && k < M;
        lo[u][k] = in ? I.box[(size_t)k * nBp + tt] : 0u;
        hi[u][k] = in ? I.box[(size_t)(M + k) * nBp + tt] : 0u;
    }
    __syncthreads();
    for (int32_t wd = w; wd < nBp / 64; wd += 4) {
        const int32_t a = wd * 64 + lane;
        const bool in = a < nB;
        bool ok[kPairWaves];
        uint32_t need[kPairWaves], apart[kPairWaves];  // (boxes that only touch: no strict inequality)
#pragma unroll
        for (int u = 0; u < kPairWaves; ++u) { ok[u] = in; need[u] = apart[u] = 0; }
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const uint32_t alo = in ? I.box[(size_t)k * nBp + a] : 0u;
            const uint32_t ahi = in ? I.box[(size_t)(M + k) * nBp + a] : 0u;
#pragma unroll
            for (int u = 0; u < kPairWaves; ++u) {
                ok[u] = ok[u] && alo <= hi[u][k];
                apart[u] |= alo ^ hi[u][k];
                need[u] |= ahi > lo[u][k] ? 1u << k : 0u;
            }
        }
        uint32_t any = 0;
#pragma unroll
        for (int u = 0; u < kPairWaves; ++u) any |= ok[u] && apart[u] != 0u ? 1u << (28 + u) : 0u;
        const uint64_t m = ballot(any != 0u);
        int32_t at = 0;
        if (lane == 0 && m) at = atomicAdd(&s_n, (int32_t)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at) + (int32_t)lanes_below(m);
        if (any) ent[at] = make_uint4((uint32_t)a | any, need[0] | need[1] << 16,
                                      need[2] | need[3] << 16, (uint32_t)tg);
    }
    __syncthreads();
    const int32_t n = s_n, items = (n + kListItem - 1) / kListItem;
    if (threadIdx.x == 0) s_base = (int32_t)atomicAdd(&I.sync->items[step], (uint32_t)items);
    __syncthreads();
    for (int32_t q = threadIdx.x; q < items * kListItem; q += 256)
        I.list[(size_t)s_base * kListItem + q] = q < n ? ent[q] : make_uint4(0u, 0u, 0u, ~0u);
}

template <int M, bool kOut, bool kMask>
__global__ __launch_bounds__(kPairWaves * kWave) void k_pairs_list(PairInst I, int32_t step) {
    __shared__ __attribute__((aligned(16))) uint32_t lt[wblk_stride(M)];
    __shared__ uint32_t oc[kOut ? kWBlk : 1];
    __shared__ uint32_t s_next;
    if (I.sc->err) return;
    const PhaseAt at = phase_at(I, step);
    const int32_t pass = at.taken;
    if (!kMask && (pass != step || at.stop)) return;  // (the last pass, which keeps masks, is next)
    I = phase_inst(I, pass);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = (int)lane_id();
    const uint32_t items = I.sync->items[pass];
    uint32_t q = blockIdx.x;
    while (q < items) {
        if (threadIdx.x == 0) s_next = gridDim.x + atomicAdd(&I.sync->next[pass], 1u);
        const uint4 e = I.list[(size_t)q * kListItem + (lane < kListItem ? lane : 0)];
        const bool in = lane < kListItem && e.w != ~0u;
        const uint32_t need = ((w & 2 ? e.z : e.y) >> (16 * (w & 1))) & 0xffffu;
        const uint64_t mine = ballot(in && ((e.x >> (28 + w)) & 1u));
        pair_blocks<M, kOut, kMask>(I, __builtin_amdgcn_readfirstlane((int)e.w),
                                    (int32_t)(e.x & 0xffffffu), need, ballot(in), mine,
                                    (int)q, lt, oc);
        __syncthreads();
        q = s_next;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// phases: the points nobody dominates are front `phase`; the others go to J in
// the same order (a block that straddled two distant chunks would meet half of
// all tiles: without the order the second pass took as long as the first).  A
// work-group takes kPhaseThreads positions, publishes how many stay, and reads
// the numbers of the work-groups before it.  One of these may not be running, for as
// long as other streams' kernels hold the CUs of its XCD (each XCD starts its own
// in order): a number that was not published after I.lookPolls looks is counted
// here, so that no work-group depends on another's start.
// ---------------------------------------------------------------------------
template <int M>
__global__ __launch_bounds__(kPhaseThreads) void k_phase(PairInst I, int32_t phase) {
    constexpr int MP = rec_stride(M);
    __shared__ uint32_t lds[kPhaseThreads / kWave + 1];
    __shared__ int32_t s_at;
    if (I.sc->err) return;
    const PhaseAt pa = phase_at(I, phase);
    if (pa.taken != phase || pa.stop) return;
    PairInst J = I;  // where the points that stay go
    if ((phase & 1) == 0) {
        J.recs = I.trec;
        J.sval = I.code;
        J.runs = I.runs2;
        J.rune = I.rune2;
        J.din = I.din2;
    }
    I = phase_inst(I, phase);
    const int32_t blk = (int32_t)blockIdx.x;
    const int32_t c0 = blk * kPhaseThreads;
    if (c0 >= I.N) return;  // (work-groups after this one return too)
    const int32_t p = c0 + (int32_t)threadIdx.x;
    const bool in = p < I.N;
    const int32_t d = in ? I.din[p] : 0;
    const uint32_t i = in ? I.sval[p] : 0u;
    const bool stays = d != 0;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(stays ? 1u : 0u, lds, &tot);
    uint32_t *cnt = I.sync->chunk[phase];
    if (threadIdx.x == 0) {
        __hip_atomic_store(&cnt[blk], 0x80000000u | tot, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        atomicAdd(&I.sync->left[phase], (int32_t)tot);
        const int32_t n = min(kPhaseThreads, I.N - c0) - (int32_t)tot;
        if (n) atomicAdd(&I.sync->lv[phase], (uint32_t)n);
        s_at = 0;
    }
    __syncthreads();
    if ((int32_t)threadIdx.x < blk) {
        uint32_t v;
        int32_t looks = 0;
        while (!((v = __hip_atomic_load(&cnt[threadIdx.x], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT)) & 0x80000000u)) {
            if (looks++ >= I.lookPolls) {  // (the degrees are this launch's input)
                const int32_t b = (int32_t)threadIdx.x * kPhaseThreads;
                v = 0;
                for (int32_t q = b; q < b + kPhaseThreads; ++q) v += I.din[q] != 0 ? 1u : 0u;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        atomicAdd(&s_at, (int32_t)(v & 0x7fffffffu));
    }
    __syncthreads();
    if (in) {
        if (I.dom_in) I.dom_in[i] = d;
        if (I.dom_out) I.dom_out[i] = I.dout[p];
        if (!stays) I.rank[i] = phase;
    }
    if (stays) {
        const int32_t q = s_at + (int32_t)ex;
        uint32_t v[MP];
#pragma unroll
        for (int k = 0; k < MP; ++k) v[k] = I.recs[(size_t)p * MP + k];
        v[M] = (uint32_t)q;
        uint4 *dst = reinterpret_cast<uint4 *>(J.recs + (size_t)q * MP);
#pragma unroll
        for (int k = 0; k < MP / 4; ++k)
            dst[k] = make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
        J.sval[q] = i;
        J.runs[q] = q - (p - I.runs[p]);  // (a run of identical rows stays whole)
        J.rune[q] = q + (I.rune[p] - p);
        J.din[q] = 0;
    }
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
template <int M>
static hipError_t launch_pairs(const PairInst &I, const RefArgs &R, bool one, uint32_t *zero,
                               int64_t nzero, const Marker &mark, hipStream_t s) {
    const unsigned nbN = (unsigned)((I.N + 255) / 256);
    if (one)
        hipLaunchKernelGGL(k_order_one<M>, dim3(1), dim3(kOrderOne), 0, s, I, R, zero, nzero);
    else
        hipLaunchKernelGGL(k_cell_sort<M>, dim3(nbN), dim3(256), 0, s, I);
    mark();
    if (I.tabs64) {
        const hipError_t e = run_build_tables(I.recs, I.N, M, I.tabs64, I.sc, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_pair_build<M, false>), dim3((unsigned)I.nB), dim3(M * kWave), 0, s, I, 0);
    const unsigned tgs = (unsigned)((I.nB + kPairWaves - 1) / kPairWaves);
    const dim3 th(kPairWaves * kWave);
    const int phases = pair_phases(I.N, M);
    if (phases == 0) {
        const int32_t G = pair_range(I.nB);
        const dim3 grid(tgs, (unsigned)((I.nB + G - 1) / G));
        if (I.dom_out)
            hipLaunchKernelGGL((k_pairs<M, true>), grid, th, 0, s, I, G);
        else
            hipLaunchKernelGGL((k_pairs<M, false>), grid, th, 0, s, I, G);
        mark();
        return run_ranks(I, 0, s);
    }
    const dim3 grid(kListGroups);
    hipLaunchKernelGGL(k_pair_list<M>, dim3(tgs), dim3(256), 0, s, I, 0);
    if (I.dom_out)
        hipLaunchKernelGGL((k_pairs_list<M, true, false>), grid, th, 0, s, I, 0);
    else
        hipLaunchKernelGGL((k_pairs_list<M, false, false>), grid, th, 0, s, I, 0);
    mark();
    for (int p = 0; p < phases; ++p) {  // (the sizes are on the device from here on)
        hipLaunchKernelGGL(k_phase<M>, dim3((unsigned)((I.N + kPhaseThreads - 1) / kPhaseThreads)),
                           dim3(kPhaseThreads), 0, s, I, p);
        hipLaunchKernelGGL((k_pair_build<M, true>), dim3((unsigned)I.nB), dim3(M * kWave), 0, s, I,
                           p + 1);
        hipLaunchKernelGGL(k_pair_list<M>, dim3(tgs), dim3(256), 0, s, I, p + 1);
        if (p + 1 < phases)
            hipLaunchKernelGGL((k_pairs_list<M, false, false>), grid, th, 0, s, I, p + 1);
        else
            hipLaunchKernelGGL((k_pairs_list<M, false, true>), grid, th, 0, s, I, p + 1);
    }
    return run_ranks(I, phases, s);
}

hipError_t run_pairs(const PairInst &I, const RefArgs &R, uint32_t *zero, int64_t nzero,
                     const Marker &mark, hipStream_t s) {
    const bool one = (int64_t)I.N * I.M <= kOrderOneKeys && R.Hpad <= kOrderOneRefs;
    if (!one) {
        const int nfill = (int)((nzero + 4 * kSplitterSample - 1) / (4 * kSplitterSample));
        const int nf = nfill < 1 ? 1 : nfill > 512 ? 512 : nfill;
        hipLaunchKernelGGL(k_pair_setup, dim3((unsigned)(I.M + 1 + nf)), dim3(kSplitterSample), 0, s, I,
                           zero, nzero, nf);
        const unsigned nbN = (unsigned)((I.N + 255) / 256);
        hipLaunchKernelGGL(k_cell_code, dim3(nbN), dim3(256), 0, s, I);
        hipLaunchKernelGGL(k_cell_scan, dim3((unsigned)(1 + (R.Hpad + 1023) / 1024)), dim3(1024), 0, s,
                           I, R);
        hipLaunchKernelGGL(k_cell_place, dim3(nbN), dim3(256), 0, s, I);
    }
    hipError_t e;
    switch (I.M) {
#define NSGA3_CASE(m) case m: e = launch_pairs<m>(I, R, one, zero, nzero, mark, s); break;
        NSGA3_CASE(2) NSGA3_CASE(3) NSGA3_CASE(4) NSGA3_CASE(5) NSGA3_CASE(6) NSGA3_CASE(7)
        NSGA3_CASE(8) NSGA3_CASE(9) NSGA3_CASE(10) NSGA3_CASE(11) NSGA3_CASE(12) NSGA3_CASE(13)
        NSGA3_CASE(14) NSGA3_CASE(15) NSGA3_CASE(16)
#undef NSGA3_CASE
        default: return hipErrorInvalidValue;
    }
    return e;
}

}  // namespace nsga3
