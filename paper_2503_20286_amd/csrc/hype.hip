// Environmental selection of TensorHypE (Sec. IV-C; Supplementary Alg. S.10,
// S.11): after the nondominated sort of the merged population (ranks r and
// the last admitted front l for a population of n), the members of F_l with
// the largest Monte Carlo hypervolume estimates fill the places left.
//
//   k = |{r <= l}| - n;  alpha_c = (1/c) prod_{i=1}^{c-1} (k - i) / (N - i)
//   f_l = the per-objective minimum over all N points, f_u = the reference
//   point, V = prod_j (f_u,j - f_l,j); sample i is S_i = f_l + U_i (f_u - f_l)
//   (U the caller's uniform draws, each sample rounded to float32 once);
//   count_i = #{p : F_p <= S_i}; HV_p = sum over the samples i that F_p
//   weakly dominates with count_i <= k of alpha_{count_i}, times V / s.
//
//  k_hv_samples  sample order keys, V, and the draws' finiteness
//  k_hv_counts   count_i: each lane probes the block tables of all points
//                (built by the dominance stage) with its samples: the members
//                with every key <= the sample's are one AND of prefix masks
//  k_hv_alpha    the alpha weights: chunked products in one work-group
//  k_hv_weights  w_i = alpha_{count_i} for 1 <= count_i <= k (else 0), and the
//                flags of those samples (compacted in order afterwards)
//  k_hv_sum      per point of r <= l: the weights of the kept samples it
//                dominates, added in float64 with their rounding errors kept, a
//                part of the samples at a time, staged through LDS
//  k_hv_keys     the parts added in order; sort keys: F_l members by descending
//                estimate (then index); flags of r < l
//  k_hv_select   the first R in that order join the selection (k_hv_pick after
//                a sort of all points for large populations)
#include <float.h>

#include "bitdom.h"
#include "kernels.h"
#include "prims.h"

namespace nsga3 {

constexpr int kHvThreads = 256;
constexpr int kHvSumChunk = 512;       // samples staged per step of k_hv_sum

struct HvState {
    double V;                           // box volume prod (f_u - f_l)
    int64_t k;                          // |S| - n
    uint32_t nrel;                      // samples with 1 <= count <= k
    uint32_t nlast;                     // members of F_l in the selection's list
};

__global__ void k_hv_samples(const float *__restrict__ U, int64_t s, int M, const float *__restrict__ vref,
                             DevScalars *sc, uint32_t *__restrict__ skeys, HvState *hs) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) {
        hs->nlast = 0u;
        double V = 1.0;
        bool ok = true;
        for (int j = 0; j < M; ++j) {
            ok = ok && isfinite(vref[j]);
            V = V * ((double)vref[j] - (double)key_to_float(sc->min_key[j]));
        }
        hs->V = V;
        if (!ok) atomicOr(&sc->err, kErrNonfiniteObj);
    }
    if (t >= s * M) return;
    const int j = (int)(t % M);
    const float u = U[t];
    if (!isfinite(u)) atomicOr(&sc->err, kErrNonfiniteObj);
    const double fl = (double)key_to_float(sc->min_key[j]);
    const float x = (float)(fl + (double)u * ((double)vref[j] - fl));
    skeys[t] = order_key(x);
}

// count_i over all points: work-group (tile group jg of kHvTiles x 512
// samples, chunk group cg of kHvChunks table chunks), one atomic per sample.
constexpr int kHvTiles = 2;
constexpr int kHvChunks = 2;

template <int M>
__global__ __launch_bounds__(kFwdThreads) void k_hv_counts(const uint32_t *__restrict__ tabs,
                                                           int32_t nblk,
                                                           const uint32_t *__restrict__ skeys,
                                                           int64_t s, int32_t *__restrict__ count,
                                                           const DevScalars *__restrict__ sc) {
    constexpr int CB = count_chunk<M>();
    constexpr int TS = blk_stride(M);
    __shared__ __attribute__((aligned(16))) uint32_t lt[CB * TS];
    if (sc->err) return;
    const int32_t nIC = (nblk + CB - 1) / CB;
    const int32_t c0 = (int32_t)blockIdx.y * kHvChunks;
    const int32_t c1 = min(c0 + kHvChunks, nIC);
    if (c0 >= nIC) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = (int)lane_id();
    uint32_t x[kHvTiles][kTJ][M];
    int32_t cnt[kHvTiles][kTJ];
#pragma unroll
    for (int t = 0; t < kHvTiles; ++t)
#pragma unroll
        for (int u = 0; u < kTJ; ++u) {
            const int64_t i = ((int64_t)blockIdx.x * kHvTiles + t) * kTileJ + w * kWave * kTJ + u * kWave + lane;
            cnt[t][u] = 0;
#pragma unroll
            for (int k = 0; k < M; ++k) x[t][u][k] = i < s ? skeys[i * M + k] : 0u;  // 0: below every key
        }
    for (int32_t c = c0; c < c1; ++c) {
        const int32_t b0 = c * CB;
        const int32_t nb = min(CB, nblk - b0);
        __syncthreads();
        stage_tables<M>(lt, tabs, b0, nb);
        __syncthreads();
        for (int32_t b = 0; b < nb; ++b) {
            const uint32_t *T = lt + b * TS;
#pragma unroll
            for (int t = 0; t < kHvTiles; ++t) {
                int ko[kTJ * M];
                uint32_t xx[kTJ * M];
                uint64_t pm[kTJ * M];
#pragma unroll
                for (int u = 0; u < kTJ; ++u)
#pragma unroll
                    for (int k = 0; k < M; ++k) {
                        ko[u * M + k] = k;
                        xx[u * M + k] = x[t][u][k];
                    }
                masks_many64<M, kTJ * M, true>(T, ko, xx, pm);
#pragma unroll
                for (int u = 0; u < kTJ; ++u) {
                    uint64_t m = ~0ull;
#pragma unroll
                    for (int k = 0; k < M; ++k) m &= pm[u * M + k];
                    cnt[t][u] += __popcll(m);
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < kHvTiles; ++t)
#pragma unroll
        for (int u = 0; u < kTJ; ++u) {
            const int64_t i = ((int64_t)blockIdx.x * kHvTiles + t) * kTileJ + w * kWave * kTJ + u * kWave + lane;
            if (i < s && cnt[t][u]) atomicAdd(&count[i], cnt[t][u]);
        }
}

// alpha_c = prod_{i<c} f_i / c with f_i = (k - i) / (N - i): thread q multiplies
// the factors of its chunk of c, a scan multiplies the chunk products, and each
// c is its chunk's prefix times its own running product.
__global__ __launch_bounds__(1024) void k_hv_alpha(int64_t N, int64_t n, const DevScalars *__restrict__ sc,
                                                   double *__restrict__ alpha, HvState *hs) {
    __shared__ double part[1024];
    if (sc->err) return;
    const int64_t k = sc->n_before + (int64_t)sc->last_front_size - n;
    if (threadIdx.x == 0) hs->k = k;
    if (k <= 0) return;
    const int64_t per = (k + blockDim.x - 1) / blockDim.x;
    const int64_t c0 = 1 + (int64_t)threadIdx.x * per;
    const int64_t c1 = c0 + per <= k + 1 ? c0 + per : k + 1;
    double p = 1.0;
    for (int64_t c = c0; c < c1; ++c)
        if (c > 1) p = p * ((double)(k - (c - 1)) / (double)(N - (c - 1)));
    part[threadIdx.x] = p;
    __syncthreads();
    if (threadIdx.x == 0) {  // exclusive product scan (1024 steps, one thread)
        double run = 1.0;
        for (unsigned q = 0; q < blockDim.x; ++q) {
            const double v = part[q];
            part[q] = run;
            run = run * v;
        }
    }
    __syncthreads();
    double q = part[threadIdx.x];
    for (int64_t c = c0; c < c1; ++c) {
        if (c > 1) q = q * ((double)(k - (c - 1)) / (double)(N - (c - 1)));
        alpha[c - 1] = q / (double)c;
    }
}

__global__ void k_hv_weights(int64_t s, const int32_t *__restrict__ count, const double *__restrict__ alpha,
                             double *__restrict__ w, uint8_t *__restrict__ flag,
                             const HvState *__restrict__ hs, const DevScalars *__restrict__ sc) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= s) return;
    const int64_t c = count[i];
    const bool keep = !sc->err && c >= 1 && c <= hs->k;
    w[i] = keep ? alpha[c - 1] : 0.0;
    flag[i] = keep ? 1 : 0;
}

// Estimates: a work-group's points (one a lane) against one part of the kept
// samples.  The additions of a point's estimate are one chain of float64
// latencies per sample, so the samples are cut into up to kHvParts parts and
// the partial sums are added in order afterwards (k_hv_keys); the cut depends
// on the number of samples alone.  N = 20k points, 10k samples, M = 3: 279 us
// in one chain over 313 waves.
constexpr int kHvParts = 8;
constexpr int kHvPartMin = kHvSumChunk;   // samples of a part, at least

// acc + x with the rounding error kept in low (x, acc >= 0; exact where acc >= x):
// another order of the samples must not lose digits against one chain.
__device__ __forceinline__ void add_comp(double &acc, double &low, double x) {
    const double s = acc + x;
    low = low + (x - (s - acc));
    acc = s;
}

static int64_t hv_part_samples(int64_t s) {
    const int64_t p = (s + kHvParts - 1) / kHvParts;
    return p < kHvPartMin ? kHvPartMin : p;
}
static int hv_parts(int64_t s) { return (int)((s + hv_part_samples(s) - 1) / hv_part_samples(s)); }

template <int M>
__global__ __launch_bounds__(kHvThreads) void k_hv_sum(const float *__restrict__ objs, int64_t N,
                                                        const int32_t *__restrict__ rank,
                                                        const uint32_t *__restrict__ skeys,
                                                        const double *__restrict__ w,
                                                        const int32_t *__restrict__ rel,
                                                        int64_t per,
                                                        const HvState *__restrict__ hs,
                                                        const DevScalars *__restrict__ sc,
                                                        double *__restrict__ part) {
    constexpr int kU = 4;  // samples whose keys are read from LDS at once
    __shared__ __attribute__((aligned(16))) uint32_t ks[M][kHvSumChunk];
    __shared__ __attribute__((aligned(16))) double ws[kHvSumChunk];
    if (sc->err) return;
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t l = sc->last_front;
    const bool mine = p < N && rank[p] <= l;
    uint32_t key[M];
#pragma unroll
    for (int k = 0; k < M; ++k) key[k] = p < N ? order_key(objs[p * M + k]) : 0xffffffffu;
    const int64_t nrel = hs->nrel;
    const int64_t b0 = (int64_t)blockIdx.y * per;
    const int64_t b1 = b0 + per < nrel ? b0 + per : nrel;
    const bool any = ballot(mine) != 0ull;
    double acc = 0.0, low = 0.0;
    for (int64_t q0 = b0; q0 < b1; q0 += kHvSumChunk) {
        const int nq = b1 - q0 < kHvSumChunk ? (int)(b1 - q0) : kHvSumChunk;
        const int nr = (nq + kU - 1) / kU * kU;
        lds_wait();
        __syncthreads();
        for (int q = threadIdx.x; q < nr; q += blockDim.x) {
            const int64_t i = q < nq ? rel[q0 + q] : -1;  // (the last few add zeros)
#pragma unroll
            for (int k = 0; k < M; ++k) ks[k][q] = i >= 0 ? skeys[i * M + k] : 0u;
            ws[q] = i >= 0 ? w[i] : 0.0;
        }
        __syncthreads();
        if (any) {
            for (int q = 0; q < nr; q += kU) {
                bool dom[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) dom[u] = true;
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(&ks[k][q]);
                    dom[0] = dom[0] & (key[k] <= v.x);
                    dom[1] = dom[1] & (key[k] <= v.y);
                    dom[2] = dom[2] & (key[k] <= v.z);
                    dom[3] = dom[3] & (key[k] <= v.w);
                }
                double a[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) a[u] = dom[u] ? ws[q + u] : 0.0;
#pragma unroll
                for (int u = 0; u < kU; ++u) add_comp(acc, low, a[u]);
            }
        }
    }
    if (mine) part[(int64_t)blockIdx.y * N + p] = acc + low;
}

// Estimates from their parts; members of F_l with their sort keys (descending
// estimate: it is >= 0, so its bits order like it), in no particular order;
// flags of r < l.  With `sorted` every point gets a key, those outside F_l
// after all others.
__global__ void k_hv_keys(int64_t N, int64_t s, int parts, const int32_t *__restrict__ rank,
                          const double *__restrict__ part, double *__restrict__ d,
                          uint64_t *__restrict__ key, uint32_t *__restrict__ val, bool sorted,
                          uint8_t *__restrict__ selflag, HvState *__restrict__ hs,
                          const DevScalars *__restrict__ sc) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool err = sc->err != 0;
    const int32_t l = sc->last_front;
    const int32_t r = i < N ? rank[i] : 0x7fffffff;
    double e = -INFINITY;
    if (!err && i < N) {
        if (r <= l) {
            double acc = part[i], low = 0.0;
            for (int q = 1; q < parts; ++q) add_comp(acc, low, part[(int64_t)q * N + i]);
            e = (acc + low) * hs->V / (double)s;
        }
        d[i] = e;
    }
    const bool last = !err && i < N && r == l;
    const uint64_t k = last ? 0x7fffffffffffffffull - (uint64_t)__double_as_longlong(e) : ~0ull;
    if (sorted) {
        if (i < N) {
            key[i] = k;
            val[i] = (uint32_t)i;
        }
    } else {
        const uint64_t m = ballot(last);
        uint32_t at = 0;
        if (m && lane_id() == 0) at = atomicAdd(&hs->nlast, (uint32_t)__popcll(m));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + lanes_below(m);
        if (last) {
            key[at] = k;
            val[at] = (uint32_t)i;
        }
    }
    if (i < N) selflag[i] = r < l ? 1 : 0;
}

// The R members of F_l with the smallest (key, index) join the selection: the
// R-th smallest key by its digits from the top, one work-group over the list
// of F_l, then (ties across the cut) the index by its digits.  Eight launches
// of a histogram and a scatter each otherwise, which stay for populations above
// kHvSelectMax.  The list is short where there are several fronts; a population
// of one front is its worst case (M = 3, by digits / by sort: 5k of N = 200k in F_l
// 3.06 / 3.17 ms; one front, N = 20k 0.31 / 0.36, 50k 0.44 / 0.45, 200k 1.20 / 0.72,
// with one member of a thread read at a time 1.48, and 2.30 / 1.59 at 250k).
constexpr int64_t kHvSelectMax = 204800;
constexpr int kHvAhead = 8;   // members of a thread that are read at once

template <typename T, typename F>
__device__ __forceinline__ T hv_digits(int nd, uint32_t n, uint32_t &need, int &sh, uint32_t *hist,
                                       uint32_t *pick, const F &get) {
    // prefix of the need-th smallest of the values that get(i, v) admits; sh:
    // bits below it (0, or more where everything with that prefix is taken)
    T prefix = 0;
    sh = 8 * nd;
    while (sh > 0) {
        for (uint32_t q = threadIdx.x; q < 256u; q += blockDim.x) hist[q] = 0u;
        lds_wait();
        __syncthreads();
        sh -= 8;
        auto tally = [&](bool in, T v) {
            in = in && (sh + 8 == 8 * nd || (T)(v >> (sh + 8)) == prefix);
            const uint32_t dg = (uint32_t)(v >> sh) & 255u;
            const uint64_t act = ballot(in);
            if (!act) return;
            // (keys share their top digits: one atomic where a wave agrees)
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)dg, __builtin_ctzll(act));
            if (ballot(in && dg == d0) == act) {
                if (lane_id() == 0) atomicAdd(&hist[d0], (uint32_t)__popcll(act));
            } else if (in) {
                atomicAdd(&hist[dg], 1u);
            }
        };
        uint32_t i0 = 0;
        for (; i0 + kHvAhead * blockDim.x <= n; i0 += kHvAhead * blockDim.x) {
            T v[kHvAhead];
            bool in[kHvAhead];
#pragma unroll
            for (int u = 0; u < kHvAhead; ++u)
                in[u] = get(i0 + (uint32_t)u * blockDim.x + threadIdx.x, v[u]);
#pragma unroll
            for (int u = 0; u < kHvAhead; ++u) tally(in[u], v[u]);
        }
        for (; i0 < n; i0 += blockDim.x) {
            const uint32_t i = i0 + threadIdx.x;
            T v = 0;
            const bool in = i < n && get(i, v);
            tally(in, v);
        }
        lds_wait();
        __syncthreads();
        if (threadIdx.x < kWave) {
            uint32_t c[4], t = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) t += c[q] = hist[threadIdx.x * 4 + q];
            uint32_t before = wave_inclusive_scan<false>(t) - t;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (before < need && need <= before + c[q]) {
                    pick[0] = threadIdx.x * 4 + q;
                    pick[1] = before;
                    pick[2] = c[q];
                }
                before += c[q];
            }
        }
        lds_wait();
        __syncthreads();
        prefix = (T)(prefix << 8) | (T)pick[0];
        need -= pick[1];
        const uint32_t c = pick[2];
        __syncthreads();
        if (c == need) break;
    }
    return prefix;
}

__global__ __launch_bounds__(1024) void k_hv_select(const uint64_t *__restrict__ key,
                                                    const uint32_t *__restrict__ val,
                                                    uint8_t *__restrict__ selflag,
                                                    const HvState *__restrict__ hs,
                                                    const DevScalars *__restrict__ sc) {
    __shared__ uint32_t hist[256];
    __shared__ uint32_t pick[3];
    if (sc->err) return;
    const uint32_t n = hs->nlast;
    const int64_t R = sc->num_from_last;
    if (R <= 0 || n == 0) return;
    uint32_t need = R < (int64_t)n ? (uint32_t)R : n;
    int sh = 0, vsh = 32;
    const uint64_t cut = hv_digits<uint64_t>(8, n, need, sh, hist, pick, [&](uint32_t i, uint64_t &v) {
        v = key[i];
        return true;
    });
    uint64_t vcut = ~0ull;
    uint32_t ties = pick[2];  // members with the cut's prefix
    __syncthreads();
    if (ties != need) {
        vcut = hv_digits<uint64_t>(4, n, need, vsh, hist, pick, [&](uint32_t i, uint64_t &v) {
            v = val[i];
            return key[i] == cut;
        });
    }
    auto mark = [&](uint64_t k, uint32_t i) {
        k >>= sh;
        if (k < cut || (k == cut && ((uint64_t)i >> vsh) <= vcut)) selflag[i] = 1;
    };
    uint32_t i0 = threadIdx.x;
    for (; i0 + (kHvAhead - 1) * blockDim.x < n; i0 += kHvAhead * blockDim.x) {
        uint64_t k[kHvAhead];
        uint32_t i[kHvAhead];
#pragma unroll
        for (int u = 0; u < kHvAhead; ++u) {
            k[u] = key[i0 + (uint32_t)u * blockDim.x];
            i[u] = val[i0 + (uint32_t)u * blockDim.x];
        }
#pragma unroll
        for (int u = 0; u < kHvAhead; ++u) mark(k[u], i[u]);
    }
    for (; i0 < n; i0 += blockDim.x) mark(key[i0], val[i0]);
}

__global__ void k_hv_pick(const uint32_t *__restrict__ val, uint8_t *__restrict__ selflag,
                          const DevScalars *__restrict__ sc) {
    if (sc->err) return;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < sc->num_from_last) selflag[val[q]] = 1;
}

__global__ void k_hv_zero(int32_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

static size_t up256(size_t b) { return (b + 255) / 256 * 256; }

size_t hype_extra_bytes(int64_t N, int M, int64_t s) {
    return up256(sizeof(HvState)) + up256(4 * (size_t)s * M) + up256(4 * (size_t)s) +
           up256(8 * (size_t)s) + up256((size_t)s) + up256(4 * (size_t)s) + up256(8 * (size_t)N) +
           up256(8 * (size_t)N) + up256(compact_temp_bytes(s));
}

hipError_t run_hype(const HypeViews &v, hipStream_t st) {
    char *w = (char *)v.extra;
    HvState *hs = (HvState *)w;
    w += up256(sizeof(HvState));
    uint32_t *skeys = (uint32_t *)w;
    w += up256(4 * (size_t)v.s * v.M);
    int32_t *count = (int32_t *)w;
    w += up256(4 * (size_t)v.s);
    double *wt = (double *)w;
    w += up256(8 * (size_t)v.s);
    uint8_t *flag = (uint8_t *)w;
    w += up256((size_t)v.s);
    int32_t *rel = (int32_t *)w;
    w += up256(4 * (size_t)v.s);
    double *alpha = (double *)w;
    w += up256(8 * (size_t)v.N);
    double *dd = v.d ? v.d : (double *)w;
    w += up256(8 * (size_t)v.N);
    uint32_t *ctemp = (uint32_t *)w;
    const int64_t N = v.N, s = v.s;
    const int M = v.M;
    hipLaunchKernelGGL(k_hv_zero, dim3((unsigned)((s + 255) / 256 < 2048 ? (s + 255) / 256 : 2048)),
                       dim3(256), 0, st, count, s);
    const int64_t sm = s * M;
    hipLaunchKernelGGL(k_hv_samples, dim3((unsigned)((sm + 255) / 256)), dim3(256), 0, st, v.U, s, M,
                       v.vref, v.sc, skeys, hs);
    const int32_t nblk = (int32_t)((N + kBlk - 1) / kBlk);
    const unsigned nTG = (unsigned)((s + (int64_t)kHvTiles * kTileJ - 1) / ((int64_t)kHvTiles * kTileJ));
    hipError_t e = hipSuccess;
    switch (M) {
#define NSGA3_CASE(m)                                                                               \
    case m: {                                                                                       \
        const int32_t nIC = (nblk + count_chunk<m>() - 1) / count_chunk<m>();                      \
        const unsigned nCG = (unsigned)((nIC + kHvChunks - 1) / kHvChunks);                        \
        hipLaunchKernelGGL(k_hv_counts<m>, dim3(nTG, nCG), dim3(kFwdThreads), 0, st, v.tabs_all,    \
                           nblk, skeys, s, count, v.sc);                                           \
        break;                                                                                      \
    }
        NSGA3_CASE(2) NSGA3_CASE(3) NSGA3_CASE(4) NSGA3_CASE(5) NSGA3_CASE(6) NSGA3_CASE(7)
        NSGA3_CASE(8) NSGA3_CASE(9) NSGA3_CASE(10) NSGA3_CASE(11) NSGA3_CASE(12) NSGA3_CASE(13)
        NSGA3_CASE(14) NSGA3_CASE(15) NSGA3_CASE(16)
#undef NSGA3_CASE
        default: return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_hv_alpha, dim3(1), dim3(1024), 0, st, N, v.n, v.sc, alpha, hs);
    const unsigned gS = (unsigned)((s + 255) / 256);
    hipLaunchKernelGGL(k_hv_weights, dim3(gS), dim3(256), 0, st, s, count, alpha, wt, flag, hs, v.sc);
    compact_flags(flag, s, rel, s, ctemp, &hs->nrel, st);
    const unsigned gN = (unsigned)((N + kHvThreads - 1) / kHvThreads);
    const int parts = hv_parts(s);
    double *part = v.part;
    switch (M) {
#define NSGA3_CASE(m)                                                                               \
    case m:                                                                                         \
        hipLaunchKernelGGL(k_hv_sum<m>, dim3(gN, (unsigned)parts), dim3(kHvThreads), 0, st, v.objs, \
                           N, v.rank, skeys, wt, rel, hv_part_samples(s), hs, v.sc, part);         \
        break;
        NSGA3_CASE(2) NSGA3_CASE(3) NSGA3_CASE(4) NSGA3_CASE(5) NSGA3_CASE(6) NSGA3_CASE(7)
        NSGA3_CASE(8) NSGA3_CASE(9) NSGA3_CASE(10) NSGA3_CASE(11) NSGA3_CASE(12) NSGA3_CASE(13)
        NSGA3_CASE(14) NSGA3_CASE(15) NSGA3_CASE(16)
#undef NSGA3_CASE
        default: return hipErrorInvalidValue;
    }
    const bool sorted = N > kHvSelectMax;
    hipLaunchKernelGGL(k_hv_keys, dim3(gN), dim3(kHvThreads), 0, st, N, s, parts, v.rank, part, dd,
                       v.skey, v.sval, sorted, v.selflag, hs, v.sc);
    if (sorted) {
        bool in_alt = false;
        radix_sort_pairs(v.skey, v.sval, v.skey_alt, v.sval_alt, N, 64, v.temp, st, &in_alt);
        hipLaunchKernelGGL(k_hv_pick, dim3(gN), dim3(kHvThreads), 0, st, in_alt ? v.sval_alt : v.sval,
                           v.selflag, v.sc);
    } else {
        hipLaunchKernelGGL(k_hv_select, dim3(1), dim3(1024), 0, st, v.skey, v.sval, v.selflag, hs,
                           v.sc);
    }
    run_compact(v.selflag, N, v.selected, v.n, v.temp, v.sc, v.info, st);
    e = hipGetLastError();
    return e;
}

}  // namespace nsga3
