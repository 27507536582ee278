// Normalisation, association, niche counting and niche-preserving selection
// on gfx950 (stages after the nondominated sort).
//
//  a4/a5  Alg. S.5: ideal point z (minimum over all points, which equals the
//         minimum over S = {rank <= l}: every minimiser of an objective is
//         dominated only by other minimisers, so one of them is nondominated),
//         extreme points by the achievement scalarising function with weights
//         1 (own axis) and 1e-6 (other axes, applied as x 1e6), hyperplane
//         intercepts from E b = 1 by Gaussian elimination with partial
//         pivoting in float64, with the nadir point as fallback.
//  a6     Eq. (10): perpendicular distance of f' = (f - z) / a to every
//         reference line.  argmin_j d_ij = argmax_j f'.rhat_j (f', rhat >= 0),
//         so candidates are screened by that dot product in float32 and the
//         survivors are re-scored in float64 with the residual form
//         ||f' - (f'.rhat) rhat||.
//  a7     Eq. (11): niche counts rho over the admitted members (rank < l) and
//         the per-reference member counts of the last front (Eq. (12)).
//  a8     Alg. S.1 inner loop, evaluated in parallel: last-front member i of
//         reference j gets the level rho_j + t_i, t_i its position among the
//         members of j ordered by (distance, index); the loop picks exactly the
//         R smallest (level, reference) pairs, found by a threshold search.
//  a9     Eq. (13): ascending indices of the selected points.
#include <float.h>

#include "kernels.h"
#include "prims.h"
#include "stage_math.h"

namespace nsga3 {

constexpr int kNormThreads = 256;
constexpr int kRankGroup = 256;                   // threads of a bucket-rank work-group
constexpr int kRankSplit = 4;                     // threads sharing one member's count
constexpr int kRankMembers = kRankGroup / kRankSplit;  // members ranked per work-group
constexpr int kNormBlocksMax = 256;

// ---------------------------------------------------------------------------
// init: clear per-call scalars and counters (fill kernels, no memset nodes)
// ---------------------------------------------------------------------------
__global__ void k_init_scalars(DevScalars *sc) { init_scalars(sc, (int)threadIdx.x); }

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

hipError_t run_init(DevScalars *sc, int32_t *zero_i32[], const int64_t zero_n[], int nzero,
                    hipStream_t s) {
    hipLaunchKernelGGL(k_init_scalars, dim3(1), dim3(64), 0, s, sc);
    for (int q = 0; q < nzero; ++q) {
        if (!zero_i32[q] || zero_n[q] <= 0) continue;
        int64_t nb = (zero_n[q] + 255) / 256;
        if (nb > 2048) nb = 2048;
        hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)nb), dim3(256), 0, s, zero_i32[q], zero_n[q], 0);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// reference directions: validity and unit vectors (float64 and float32)
// ---------------------------------------------------------------------------
__global__ void k_refs(RefArgs R, int M, DevScalars *__restrict__ sc) {
    reference_item(R, M, (int)(blockIdx.x * blockDim.x + threadIdx.x), sc);
}

__device__ __forceinline__ double ideal(const DevScalars *sc, int k) {
    return (double)key_to_float(sc->min_key[k]);
}

// ---------------------------------------------------------------------------
// a4: extreme-point partials per work-group (ASF argmin per axis) and nadir
// partials; the last work-group to finish takes a5: reduces the partials,
// builds E, solves E b = 1 (intercepts / fallback).
// ---------------------------------------------------------------------------
// (value, index) minimum and maximum over a wave.
__device__ __forceinline__ void fold_extreme(double &b, int32_t &bi, double &nd) {
    for (int o = 32; o > 0; o >>= 1) {
        const double ob = __shfl_xor(b, o, 64);
        const int32_t oi = __shfl_xor(bi, o, 64);
        if (ob < b || (ob == b && oi < bi)) { b = ob; bi = oi; }
        const double on = __shfl_xor(nd, o, 64);
        nd = on > nd ? on : nd;
    }
}

template <int M>
__global__ __launch_bounds__(kNormThreads) void k_extreme(
    const float *__restrict__ objs, int64_t N, const int32_t *__restrict__ rank,
    DevScalars *__restrict__ sc, double *p_asf, int32_t *p_idx, double *p_nad) {
    constexpr int kW = kNormThreads / kWave;
    __shared__ double s_asf[kW][M], s_nad[kW][M];
    __shared__ int32_t s_idx[kW][M];
    __shared__ int32_t s_e[M];
    __shared__ double s_nadir[M];
    __shared__ uint32_t s_last;
    if (sc->err) return;
    const int32_t l = sc->last_front;
    double z[M], best[M], nad[M];
    int32_t bidx[M];
#pragma unroll
    for (int k = 0; k < M; ++k) {
        z[k] = ideal(sc, k);
        best[k] = DBL_MAX;
        bidx[k] = 0x7fffffff;
        nad[k] = 0.0;
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
        if (rank[i] > l) continue;
        double g[M];
#pragma unroll
        for (int k = 0; k < M; ++k) g[k] = (double)objs[i * M + k] - z[k];
        asf_fold<M>(g, M, (int32_t)i, best, bidx, nad);
    }
    const int w = threadIdx.x / kWave;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        fold_extreme(best[j], bidx[j], nad[j]);
        if (lane_id() == 0) { s_asf[w][j] = best[j]; s_idx[w][j] = bidx[j]; s_nad[w][j] = nad[j]; }
    }
    __syncthreads();
    if ((int)threadIdx.x < M) {
        const int j = threadIdx.x;
        double b = s_asf[0][j];
        int32_t bi = s_idx[0][j];
        double nd = s_nad[0][j];
        for (int q = 1; q < kW; ++q) {
            if (s_asf[q][j] < b || (s_asf[q][j] == b && s_idx[q][j] < bi)) { b = s_asf[q][j]; bi = s_idx[q][j]; }
            nd = s_nad[q][j] > nd ? s_nad[q][j] : nd;
        }
        p_asf[blockIdx.x * M + j] = b;
        p_idx[blockIdx.x * M + j] = bi;
        p_nad[blockIdx.x * M + j] = nd;
        __threadfence();
    }
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&sc->ext_done, 1u) + 1u == gridDim.x ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    __threadfence();  // every work-group's partials
    // a wave folds every kW-th axis
    for (int j = w; j < M; j += kW) {
        double b = DBL_MAX, nd = 0.0;
        int32_t bi = 0x7fffffff;
        for (int q = (int)lane_id(); q < (int)gridDim.x; q += kWave) {
            const double x = __hip_atomic_load(&p_asf[q * M + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int32_t xi = __hip_atomic_load(&p_idx[q * M + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const double xn = __hip_atomic_load(&p_nad[q * M + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (x < b || (x == b && xi < bi)) { b = x; bi = xi; }
            nd = xn > nd ? xn : nd;
        }
        fold_extreme(b, bi, nd);
        if (lane_id() == 0) { s_e[j] = bi; s_nadir[j] = nd; }
    }
    __syncthreads();
    if (w != 0) return;
    double a[M];
    const int fb = solve_intercepts_wave<M>(objs, s_e, s_nadir, z, a);
    if (lane_id() != 0) return;
    for (int k = 0; k < M; ++k) {
        sc->z[k] = z[k];
        sc->a[k] = a[k];
    }
    sc->fallback = fb;
}

// ---------------------------------------------------------------------------
// a6/a7: association (float32 screening, float64 re-scoring) and counts.
// ---------------------------------------------------------------------------
// References that pass the screen of a lane's point wait in a list of up to
// four (16 bits each) and are re-scored together: a wave then goes through the
// float64 distance as often as its busiest lane needs it, not once for every
// reference that some lane needs (N = 200k, M = 5, 210 references: 53 us).
// The two smallest distances and the lowest index of the smallest do not
// depend on the order.
template <int M>
struct Rescore {
    double d1 = DBL_MAX, d2 = DBL_MAX;
    int32_t best = 0;
    uint64_t list = 0;
    int n = 0;
    __device__ __forceinline__ void add(bool pass, int j) {
        if (pass) {
            list = list << 16 | (uint64_t)j;
            ++n;
        }
    }
    __device__ __forceinline__ bool full() const { return ballot(n == 4) != 0ull; }
    __device__ __forceinline__ void run(const double (&fp)[M], const double *__restrict__ rhat64) {
        while (ballot(n > 0)) {
            if (n > 0) {
                const int32_t j = (int32_t)(list & 0xffffu);
                list >>= 16;
                --n;
                const double d = line_distance<M>(fp, rhat64 + (int64_t)j * M);
                if (d < d1 || (d == d1 && j < best)) { d2 = d1; d1 = d; best = j; }
                else if (d < d2) { d2 = d; }
            }
        }
    }
    // with the lane that holds other references of the same point
    __device__ __forceinline__ void merge(int o) {
        const double e1 = __shfl_xor(d1, o, 64), e2 = __shfl_xor(d2, o, 64);
        const int32_t eb = __shfl_xor(best, o, 64);
        if (e1 < d1 || (e1 == d1 && eb < best)) {
            d2 = fmin(d1, e2);
            d1 = e1;
            best = eb;
        } else {
            d2 = fmin(d2, e1);
        }
    }
};

// S adjacent lanes share a point, each with every S-th reference, which are
// staged in LDS (one lane a point through scalar loads: 230 us instead of 152 at N =
// 200k, M = 3, 2000 references, 47.8 and 46.7 at M = 5, 200).
constexpr int kAssocFloats = 4096;

template <int M, int S>
__global__ __launch_bounds__(kNormThreads) void k_associate(
    const float *__restrict__ objs, int64_t N, const int32_t *__restrict__ rank,
    const double *__restrict__ rhat64, const float *__restrict__ rhat32, int H,
    int32_t *__restrict__ niche, float *__restrict__ dist, double *__restrict__ dist64,
    int32_t *__restrict__ rho, int32_t *__restrict__ bcount, uint8_t *__restrict__ selflag,
    DevScalars *__restrict__ sc) {
    constexpr int kRefs = kAssocFloats / M / S * S;  // references staged at once
    __shared__ int32_t hist[2 * kLdsNicheRefs];
    __shared__ __attribute__((aligned(16))) float lr[kRefs * M];
    if (sc->err) return;
    const int32_t l = sc->last_front;
    const int sub = S > 1 ? (int)threadIdx.x % S : 0;
    const int64_t i = (int64_t)blockIdx.x * (kNormThreads / S) + (int)threadIdx.x / S;
    const int32_t r = i < N ? rank[i] : 0x7fffffff;
    const bool mine = r <= l && i < N;
    const bool any = ballot(mine) != 0ull;
    double fp[M];
    float y[M];
    float l1 = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) { fp[k] = 0.0; y[k] = 0.0f; }
    if (mine) l1 = normalise_point<M>(objs + i * M, sc->z, sc->a, fp, y);
    auto stage = [&](int c0) {
        const int n = (H - c0 < kRefs ? H - c0 : kRefs) * M;
        __syncthreads();
        for (int q = threadIdx.x; q < n; q += kNormThreads) lr[q] = rhat32[(int64_t)c0 * M + q];
        __syncthreads();
    };
    float smax = -FLT_MAX;
    for (int c0 = 0; c0 < H; c0 += kRefs) {
        stage(c0);
        const int n = H - c0 < kRefs ? H - c0 : kRefs;
        if (any) {
            int j = sub;
            for (; j + 3 * S < n; j += 4 * S) {
                float s4[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    s4[u] = screen_dot<M>(y, lr + (j + u * S) * M);
                smax = fmaxf(smax, fmaxf(fmaxf(s4[0], s4[1]), fmaxf(s4[2], s4[3])));
            }
            for (; j < n; j += S)
                smax = fmaxf(smax, screen_dot<M>(y, lr + j * M));
        }
    }
    for (int o = 1; o < S; o <<= 1) smax = fmaxf(smax, __shfl_xor(smax, o, 64));
    const float thr = smax - fp32_band<M>(l1);
    Rescore<M> R;
    for (int c0 = 0; c0 < H; c0 += kRefs) {
        if (H > kRefs) stage(c0);
        const int n = H - c0 < kRefs ? H - c0 : kRefs;
        if (any) {
            int jb = 0;
            for (; jb + 4 * S <= n; jb += 4 * S) {  // (four in a row: their loads are one)
                bool pass[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = jb + u * S + sub;
                    const float s = screen_dot<M>(y, lr + j * M);
                    pass[u] = mine && !(s < thr);
                }
                if (!ballot(pass[0] || pass[1] || pass[2] || pass[3])) continue;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    R.add(pass[u], c0 + jb + u * S + sub);
                    if (R.full()) R.run(fp, rhat64);
                }
            }
            for (; jb < n; jb += S) {
                const int j = jb + sub, jc = j < n ? j : n - 1;
                const float s = screen_dot<M>(y, lr + jc * M);
                R.add(mine && j < n && !(s < thr), c0 + j);
                if (R.full()) R.run(fp, rhat64);
            }
        }
    }
    R.run(fp, rhat64);
    for (int o = 1; o < S; o <<= 1) R.merge(o);
    int cls = -1;
    if (sub == 0) {
        if (mine) {
            niche[i] = R.best;
            if (dist) dist[i] = (float)R.d1;
            dist64[i] = R.d1;
            if (near_tie(R.d1, R.d2)) atomicAdd(&sc->near_ties, 1);
            cls = r < l ? 0 : 1;
            selflag[i] = r < l ? 1 : 0;
        } else if (i < N) {
            niche[i] = -1;
            if (dist) dist[i] = -1.0f;
            dist64[i] = -1.0;
            selflag[i] = 0;
        }
    }
    niche_count_block(H, cls, R.best, rho, bcount, hist);
}

// ---------------------------------------------------------------------------
// a6/a7, matrix-core form: the screening dot products s = y . rhat are one
// bfloat16 MFMA per 32 references x 32 points (float32 accumulate); refs are
// the A operand (rows), points the B operand (columns), so each lane holds one
// point (column l % 32) and 16 of the 32 references of the tile.  The band
// covers the bfloat16 rounding of both operands; survivors are re-scored in
// float64 exactly as in the float32 form.
// ---------------------------------------------------------------------------
typedef float mfma_f16v __attribute__((ext_vector_type(16)));
typedef short mfma_s4v __attribute__((ext_vector_type(4)));
typedef __bf16 mfma_b8v __attribute__((ext_vector_type(8)));

template <int KP>
struct BfOperand;
template <>
struct BfOperand<8> {
    using T = mfma_s4v;  // 4 bf16 per lane (k = 4 * (lane / 32) + v)
    static __device__ __forceinline__ mfma_f16v mma(T a, T b, mfma_f16v c) {
        return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ void set(T &x, int v, uint16_t bits) { x[v] = (short)bits; }
    static constexpr int kPerLane = 4;
};
template <>
struct BfOperand<16> {
    using T = mfma_b8v;  // 8 bf16 per lane (k = 8 * (lane / 32) + v)
    static __device__ __forceinline__ mfma_f16v mma(T a, T b, mfma_f16v c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ void set(T &x, int v, uint16_t bits) {
        x[v] = __builtin_bit_cast(__bf16, bits);
    }
    static constexpr int kPerLane = 8;
};

template <int M>
__global__ __launch_bounds__(256) void k_associate_bf16(
    const float *__restrict__ objs, int64_t N, const int32_t *__restrict__ rank,
    const double *__restrict__ rhat64, const uint16_t *__restrict__ rhat16, int H,
    int32_t *__restrict__ niche, float *__restrict__ dist, double *__restrict__ dist64,
    int32_t *__restrict__ rho, int32_t *__restrict__ bcount, uint8_t *__restrict__ selflag,
    DevScalars *__restrict__ sc) {
    constexpr int KP = M <= 8 ? 8 : 16;
    using Op = BfOperand<KP>;
    constexpr int KL = Op::kPerLane;
    __shared__ int32_t hist[2 * kLdsNicheRefs];
    if (sc->err) return;
    const int32_t l = sc->last_front;
    const int lane = (int)lane_id();
    const int half = lane >> 5;                       // which k-slice / row half this lane holds
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t i = wave * 32 + (lane & 31);        // this lane's point (shared with lane ^ 32)
    const bool inrange = i < N;
    const int32_t r = inrange ? rank[i] : 0x7fffffff;
    const bool active = inrange && r <= l;
    double fp[M];
    double mx = 0.0;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        fp[k] = active ? ((double)objs[i * M + k] - sc->z[k]) / sc->a[k] : 0.0;
        mx = fp[k] > mx ? fp[k] : mx;
    }
    float y[M];
    float n2 = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        y[k] = mx > 0.0 ? (float)(fp[k] / mx) : 0.0f;
        n2 = __fmaf_rn(y[k], y[k], n2);
    }
    // B operand: this lane's point, k-slice [KL * half, KL * half + KL)
    typename Op::T bop;
#pragma unroll
    for (int v = 0; v < KL; ++v) {
        const int k = KL * half + v;
        float val = 0.0f;
#pragma unroll
        for (int q = 0; q < M; ++q)
            if (q == k) val = y[q];
        Op::set(bop, v, bf16_rne(val));
    }
    const int ntiles = (H + 31) / 32;
    float smax = -FLT_MAX;
    for (int tl = 0; tl < ntiles; ++tl) {
        const typename Op::T aop = *reinterpret_cast<const typename Op::T *>(
            rhat16 + ((int64_t)(tl * 32 + (lane & 31)) * KP + KL * half));
        mfma_f16v acc = {};
        acc = Op::mma(aop, bop, acc);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int j = tl * 32 + 8 * (v / 4) + 4 * half + (v % 4);
            if (j < H) smax = acc[v] > smax ? acc[v] : smax;
        }
    }
    smax = fmaxf(smax, __shfl_xor(smax, 32, 64));
    // |s_bf16 - s| <= (2 u + u^2) ||y||_2 + float32 rounding, u = 2^-8; doubled
    const float band = 2.0f * 1.01f * (0.0078125f + 0.000244f) * sqrtf(n2) + 1e-30f;
    const float thr = smax - band;
    Rescore<M> R;
    R.best = 0x7fffffff;
    for (int tl = 0; tl < ntiles; ++tl) {
        const typename Op::T aop = *reinterpret_cast<const typename Op::T *>(
            rhat16 + ((int64_t)(tl * 32 + (lane & 31)) * KP + KL * half));
        mfma_f16v acc = {};
        acc = Op::mma(aop, bop, acc);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int j = tl * 32 + 8 * (v / 4) + 4 * half + (v % 4);
            R.add(active && j < H && !(acc[v] < thr), j);
            if (R.full()) R.run(fp, rhat64);
        }
    }
    R.run(fp, rhat64);
    R.merge(32);  // the lane with the other 16 references of every tile
    const double d1 = R.d1, d2 = R.d2;
    const int32_t best = R.best;
    int cls = -1;
    if (inrange && half == 0) {
        if (!active) {
            niche[i] = -1;
            if (dist) dist[i] = -1.0f;
            dist64[i] = -1.0;
            selflag[i] = 0;
        } else {
            niche[i] = best;
            if (dist) dist[i] = (float)d1;
            dist64[i] = d1;
            if (near_tie(d1, d2)) atomicAdd(&sc->near_ties, 1);
            cls = r < l ? 0 : 1;
            selflag[i] = r < l ? 1 : 0;
        }
    }
    niche_count_block(H, cls, best, rho, bcount, hist);
}

// ---------------------------------------------------------------------------
// a8 plan: bucket offsets of the last front by reference, and the selection
// threshold.  For threshold V, C(V) = sum_j clamp(V - rho_j, 0, b_j) members
// have level < V.  V* = max{V : C(V) <= R}; the remaining R - C(V*) picks are
// the level-V* members of the lowest-indexed references.  One block.
// ---------------------------------------------------------------------------
struct NicheLds {
    static constexpr int kRefs = 4096;
    uint32_t scan[17];
    int64_t red[16];
    int64_t vmax, V;
    int32_t thr;
    int32_t rho[kRefs], bc[kRefs];
};

__device__ __forceinline__ void niche_plan_item(int H, const int32_t *rho, const int32_t *bcount,
                                                int32_t *bstart, int32_t *bcursor, int32_t *gstart,
                                                DevScalars *sc, NicheLds &W) {
    uint32_t *lds = W.scan;
    int64_t *red = W.red;
    const int64_t R = sc->num_from_last;
    // bucket starts (exclusive scan of bcount), chunked by blockDim
    uint32_t run = 0, grun = 0;
    int64_t vmax = 0;
    for (int base = 0; base < H; base += blockDim.x) {
        const int j = base + threadIdx.x;
        const uint32_t v = j < H ? (uint32_t)bcount[j] : 0u;
        if (j < H) {
            const int64_t top = (int64_t)rho[j] + bcount[j];
            vmax = top > vmax ? top : vmax;
        }
        uint32_t tot, gtot;
        const uint32_t ex = block_exclusive_scan(v, lds, &tot);
        const uint32_t gex = block_exclusive_scan((v + kRankMembers - 1) / kRankMembers, lds, &gtot);
        if (j < H) {
            bstart[j] = (int32_t)(run + ex);
            bcursor[j] = (int32_t)(run + ex);
            gstart[j] = (int32_t)(grun + gex);
        }
        run += tot;
        grun += gtot;
    }
    if (threadIdx.x == 0) {
        bstart[H] = (int32_t)run;
        gstart[H] = (int32_t)grun;
    }
    vmax = wave_max(vmax);
    if (lane_id() == 0) red[threadIdx.x / kWave] = vmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t m = 0;
        for (unsigned q = 0; q < blockDim.x / kWave; ++q) m = red[q] > m ? red[q] : m;
        W.vmax = m;
    }
    __syncthreads();
    // binary search for V* in [0, vmax]: C is non-decreasing, C(0) = 0 <= R;
    // the counts are read from LDS when they fit (one global read each, not
    // one per search step)
    const int32_t *rho_r = rho, *bc_r = bcount;
    if (H <= NicheLds::kRefs) {
        for (int j = threadIdx.x; j < H; j += blockDim.x) {
            W.rho[j] = rho[j];
            W.bc[j] = bcount[j];
        }
        __syncthreads();
        rho_r = W.rho;
        bc_r = W.bc;
    }
    // (one wave searches: no block barriers inside the loop)
    if (threadIdx.x < kWave) {
        int64_t lo = 0, hi = W.vmax;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            int64_t c = 0;
            for (int j = threadIdx.x; j < H; j += kWave) {
                int64_t t = mid - rho_r[j];
                t = t < 0 ? 0 : t;
                c += t < bc_r[j] ? t : bc_r[j];
            }
            c = wave_sum(c);
            if (c <= R) lo = mid; else hi = mid - 1;
        }
        if (threadIdx.x == 0) W.V = lo;
    }
    __syncthreads();
    const int64_t V = W.V;
    int64_t cV = 0;
    for (int j = threadIdx.x; j < H; j += blockDim.x) {
        int64_t t = V - rho[j];
        t = t < 0 ? 0 : t;
        cV += t < bcount[j] ? t : bcount[j];
    }
    cV = wave_sum(cV);
    __syncthreads();
    if (lane_id() == 0) red[threadIdx.x / kWave] = cV;
    __syncthreads();
    int64_t CV = 0;
    for (unsigned q = 0; q < blockDim.x / kWave; ++q) CV += red[q];
    const int64_t rem = R - CV;  // picks at level V, lowest references first
    // reference threshold: the rem-th reference (ascending) with a member at level V
    int32_t thr = 0;
    uint32_t seen = 0;
    if (threadIdx.x == 0) W.thr = (rem <= 0) ? 0 : H;
    __syncthreads();
    if (rem > 0) {
        for (int base = 0; base < H; base += blockDim.x) {
            const int j = base + threadIdx.x;
            const uint32_t has = (j < H && rho[j] <= V && V < (int64_t)rho[j] + bcount[j]) ? 1u : 0u;
            uint32_t tot;
            const uint32_t ex = block_exclusive_scan(has, lds, &tot);
            if (has && (int64_t)(seen + ex) == rem - 1) W.thr = j + 1;
            seen += tot;
            __syncthreads();
            if ((int64_t)seen >= rem) break;
        }
    }
    __syncthreads();
    thr = W.thr;
    if (threadIdx.x == 0) {
        sc->level_V = (int32_t)V;
        sc->ref_thr = thr;
    }
}

__global__ __launch_bounds__(1024) void k_niche_plan(int H, const int32_t *__restrict__ rho,
                                                     const int32_t *__restrict__ bcount,
                                                     int32_t *__restrict__ bstart,
                                                     int32_t *__restrict__ bcursor,
                                                     int32_t *__restrict__ gstart,
                                                     DevScalars *__restrict__ sc) {
    __shared__ NicheLds W;
    if (sc->err) return;
    niche_plan_item(H, rho, bcount, bstart, bcursor, gstart, sc, W);
}

// last-front members -> reference buckets (order inside a bucket is arbitrary)
__global__ __launch_bounds__(256) void k_bucket_scatter(int64_t N, int H,
                                                        const int32_t *__restrict__ rank,
                                                        const int32_t *__restrict__ niche,
                                                        const double *__restrict__ dist64,
                                                        int32_t *__restrict__ bcursor,
                                                        double *__restrict__ bd,
                                                        int32_t *__restrict__ bi,
                                                        const DevScalars *__restrict__ sc) {
    __shared__ int32_t cnt[kLdsNicheRefs];
    if (sc->err) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool member = i < N && rank[i] == sc->last_front;
    const int32_t b = member ? niche[i] : 0;
    const int32_t slot = bucket_slot_block(H, member, b, bcursor, cnt);
    if (!member) return;
    bd[slot] = dist64[i];
    bi[slot] = (int32_t)i;
}

// t_i = #members of the same reference with smaller (distance, index); pick
// when (rho + t, reference) is below the threshold.  Work-group g ranks
// kRankMembers members of one bucket (gstart maps groups to buckets) against
// the whole bucket, staged through LDS; kRankSplit adjacent lanes share a
// member, each counting every kRankSplit-th bucket entry.
__global__ __launch_bounds__(kRankGroup) void k_bucket_rank(int H, const int32_t *__restrict__ rho,
                                                            const int32_t *__restrict__ bstart,
                                                            const int32_t *__restrict__ gstart,
                                                            const double *__restrict__ bd,
                                                            const int32_t *__restrict__ bi,
                                                            uint8_t *__restrict__ selflag,
                                                            const DevScalars *__restrict__ sc) {
    constexpr int kChunk = 2048;
    __shared__ double sd[kChunk];
    __shared__ int32_t si[kChunk];
    if (sc->err) return;
    const int32_t g = blockIdx.x;
    if (g >= gstart[H]) return;
    int32_t lo = 0, hi = H - 1;  // the bucket j with gstart[j] <= g < gstart[j + 1]
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (gstart[mid] <= g) lo = mid; else hi = mid - 1;
    }
    const int32_t j = lo;
    const int32_t b0 = bstart[j], b1 = bstart[j + 1];
    const int32_t s = b0 + (g - gstart[j]) * kRankMembers + (int32_t)threadIdx.x / kRankSplit;
    const int32_t sub = (int32_t)threadIdx.x % kRankSplit;
    const bool mine = s < b1;
    const double d = mine ? bd[s] : 0.0;
    const int32_t i = mine ? bi[s] : 0;
    int32_t t = 0;
    for (int32_t c0 = b0; c0 < b1; c0 += kChunk) {
        const int32_t c1 = min(c0 + kChunk, b1);
        __syncthreads();
        for (int32_t q = c0 + (int32_t)threadIdx.x; q < c1; q += kRankGroup) {
            sd[q - c0] = bd[q];
            si[q - c0] = bi[q];
        }
        __syncthreads();
        if (mine) {
            const int32_t n = c1 - c0;
#pragma unroll 4
            for (int32_t m = sub; m < n; m += kRankSplit)
                t += (sd[m] < d || (sd[m] == d && si[m] < i)) ? 1 : 0;
        }
    }
    for (int o = 1; o < kRankSplit; o <<= 1) t += __shfl_xor(t, o, 64);  // the member's lanes
    if (!mine || sub != 0) return;
    const int64_t lev = (int64_t)rho[j] + t;
    const int64_t V = sc->level_V;
    if (lev < V || (lev == V && j < sc->ref_thr)) selflag[i] = 1;
}

__device__ __forceinline__ void finalize_item(nsga3_info *info, int64_t K, int64_t n_selected,
                                              const DevScalars *__restrict__ sc) {
    uint32_t e = sc->err;
    if (e == 0 && n_selected != K) e |= kErrInternal;
    nsga3_info v;
    v.status = e == 0 ? NSGA3_OK
               : (e & (kErrNonfiniteObj | kErrBadRef)) ? NSGA3_E_NONFINITE
                                                       : NSGA3_E_HIP;
    v.last_front = sc->last_front;
    v.num_fronts = sc->num_fronts;
    v.last_front_size = sc->last_front_size;
    v.num_from_last = (int32_t)sc->num_from_last;
    v.intercept_fallback = sc->fallback;
    v.near_ties = sc->near_ties;
    v.reserved = (int32_t)e;
    *info = v;
}

__global__ void k_finalize(nsga3_info *info, int64_t K, const DevScalars *__restrict__ sc) {
    if (threadIdx.x == 0) finalize_item(info, K, sc->n_selected, sc);
}

// The indices of the set flags (0 / 1, 16-byte aligned), at most cap of them,
// and the call's info, by one work-group.
__device__ __forceinline__ void compact_item(const uint8_t *flag, int64_t N, int32_t *out,
                                             int64_t cap, uint32_t *lds, DevScalars *sc,
                                             nsga3_info *info) {
    uint32_t base = 0;
    for (int64_t c0 = 0; c0 < N; c0 += 16 * (int64_t)blockDim.x) {
        const int64_t p = c0 + 16 * (int64_t)threadIdx.x;
        uint32_t v[4] = {0, 0, 0, 0};
        if (p + 16 <= N) {
            const uint4 f = *reinterpret_cast<const uint4 *>(flag + p);
            v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
        } else {
            for (int q = 0; q < 16; ++q)
                if (p + q < N) v[q / 4] |= (uint32_t)flag[p + q] << (8 * (q % 4));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] &= 0x01010101u;
        const uint32_t n = (uint32_t)(__popc(v[0]) + __popc(v[1]) + __popc(v[2]) + __popc(v[3]));
        uint32_t tot;
        uint32_t at = base + block_exclusive_scan(n, lds, &tot);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            for (uint32_t w = v[q]; w; w &= w - 1u) {
                if ((int64_t)at < cap) out[at] = (int32_t)(p + 4 * q + __builtin_ctz(w) / 8);
                ++at;
            }
        base += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sc->n_selected = base;
        if (info) finalize_item(info, cap, base, sc);
    }
}

__global__ __launch_bounds__(1024) void k_compact_one(const uint8_t *__restrict__ flag, int64_t N,
                                                      int32_t *__restrict__ out, int64_t cap,
                                                      DevScalars *__restrict__ sc,
                                                      nsga3_info *__restrict__ info) {
    __shared__ uint32_t lds[17];
    compact_item(flag, N, out, cap, lds, sc, info);
}

// Small problems: plan, buckets, picks, compaction and info by one work-group,
// which keeps the last front's members and the flags in LDS.  A member counts
// its bucket alone, so one reference that holds all of N = 1024 members costs
// 1024 steps (about 9 us); seven launches are at least 30 us.
constexpr int kNicheOne = 1024;
constexpr int kNicheOneRefs = kLdsNicheRefs;

__global__ __launch_bounds__(1024) void k_niche_one(int N, int H, const int32_t *rank,
                                                    const int32_t *niche, const double *dist64,
                                                    const int32_t *rho, const int32_t *bcount,
                                                    int32_t *bstart, int32_t *bcursor,
                                                    int32_t *gstart, const uint8_t *selflag,
                                                    int32_t *out, int64_t K, DevScalars *sc,
                                                    nsga3_info *info) {
    __shared__ NicheLds W;
    __shared__ int32_t s_cur[kNicheOneRefs];
    __shared__ double s_d[kNicheOne];
    __shared__ int32_t s_i[kNicheOne];
    __shared__ __attribute__((aligned(16))) uint8_t s_f[kNicheOne];
    const int t = (int)threadIdx.x;
    s_f[t] = 0;
    __syncthreads();
    if (!sc->err) {
        niche_plan_item(H, rho, bcount, bstart, bcursor, gstart, sc, W);
        __syncthreads();
        for (int j = t; j < H; j += kNicheOne) s_cur[j] = bstart[j];
        __syncthreads();
        const bool in = t < N;
        const bool member = in && rank[t] == sc->last_front;
        const int32_t j = member ? niche[t] : 0;
        const double d = member ? dist64[t] : 0.0;
        if (in) s_f[t] = selflag[t];
        if (member) {
            const int32_t slot = atomicAdd(&s_cur[j], 1);
            s_d[slot] = d;
            s_i[slot] = t;
        }
        __syncthreads();
        if (member) {
            int32_t n = 0;
            const int32_t b1 = bstart[j + 1];
            for (int32_t m = bstart[j]; m < b1; ++m)
                n += (s_d[m] < d || (s_d[m] == d && s_i[m] < t)) ? 1 : 0;
            const int64_t lev = (int64_t)rho[j] + n;
            const int64_t V = sc->level_V;
            if (lev < V || (lev == V && j < sc->ref_thr)) s_f[t] = 1;
        }
        __syncthreads();
    }
    compact_item(s_f, N, out, K, W.scan, sc, info);
}

// Up to this many flags one work-group compacts them: 16 bytes a thread and
// step, where counts, scan, write and info are four launches.
constexpr int64_t kCompactOne = 65536;

// ---------------------------------------------------------------------------
// One-shot niche selection (Sec. IV-A.5; the niche-selection steps of
// Alg. S.4 and the Update-Rank of Alg. S.6): instead of admitting last-front
// members one at a time, every reference with no admitted member (rho_j = 0)
// that has last-front members admits its closest one (distance, then index)
// at once.  With |E| such picks and R places left, a shortfall R > |E| is
// filled with the R - |E| lowest-index unpicked last-front members, a surplus
// keeps the R lowest-index picks.  On the shuffled population the paper
// takes as input, index order is a random order, so both fill rules are the
// random choices the algorithm makes.
// selflag values on entry: 1 admitted (rank < l), 0 otherwise; the picks are
// marked 2 by k_oneshot_pick, and k_oneshot_apply leaves 0 / 1 everywhere.
// ---------------------------------------------------------------------------
constexpr int kOsTile = 2048;   // indices per count / apply work-group (8 x 256)

// One wave per reference: the closest member of an empty niche's bucket.
__global__ __launch_bounds__(256) void k_oneshot_pick(int H, const int32_t *__restrict__ rho,
                                                      const int32_t *__restrict__ bstart,
                                                      const double *__restrict__ bd,
                                                      const int32_t *__restrict__ bi,
                                                      uint8_t *__restrict__ selflag,
                                                      const DevScalars *__restrict__ sc) {
    if (sc->err) return;
    const int j = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (j >= H || rho[j] != 0) return;
    const int32_t b0 = bstart[j], b1 = bstart[j + 1];
    if (b1 <= b0) return;
    double d = DBL_MAX;
    int32_t i = INT32_MAX;
    for (int32_t q = b0 + (int32_t)lane_id(); q < b1; q += kWave) {
        const double dq = bd[q];
        const int32_t iq = bi[q];
        if (dq < d || (dq == d && iq < i)) { d = dq; i = iq; }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double dq = __shfl_xor(d, o, 64);
        const int32_t iq = __shfl_xor(i, o, 64);
        if (dq < d || (dq == d && iq < i)) { d = dq; i = iq; }
    }
    if (lane_id() == 0) selflag[i] = 2;
}

// Per tile of kOsTile indices: number of picks (flag 2) and of unpicked
// last-front members, in cnt[0 .. nb) and cnt[nbp .. nbp + nb).
__global__ __launch_bounds__(256) void k_oneshot_count(int64_t N, const int32_t *__restrict__ rank,
                                                       const uint8_t *__restrict__ selflag,
                                                       uint32_t *__restrict__ cnt, int64_t nbp,
                                                       const DevScalars *__restrict__ sc) {
    __shared__ uint32_t red[2][4];
    if (sc->err) return;
    const int32_t l = sc->last_front;
    const int64_t base = (int64_t)blockIdx.x * kOsTile;
    uint32_t cp = 0, cq = 0;
#pragma unroll
    for (int it = 0; it < kOsTile / 256; ++it) {
        const int64_t p = base + it * 256 + threadIdx.x;
        if (p < N) {
            const uint8_t f = selflag[p];
            cp += f == 2 ? 1u : 0u;
            cq += (f != 2 && rank[p] == l) ? 1u : 0u;
        }
    }
    cp = wave_sum(cp);
    cq = wave_sum(cq);
    if (lane_id() == 0) {
        red[0][threadIdx.x / kWave] = cp;
        red[1][threadIdx.x / kWave] = cq;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        cnt[blockIdx.x] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        cnt[nbp + blockIdx.x] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
}

// Final flags: a pick stays when R >= |E| or fewer than R picks precede it; an
// unpicked last-front member is added when fewer than R - |E| of them precede
// it.  off holds the exclusive tile prefixes of both counts (as cnt above);
// totals[0] = |E|.
__global__ __launch_bounds__(256) void k_oneshot_apply(int64_t N, const int32_t *__restrict__ rank,
                                                       uint8_t *__restrict__ selflag,
                                                       const uint32_t *__restrict__ off, int64_t nbp,
                                                       const uint32_t *__restrict__ totals,
                                                       const DevScalars *__restrict__ sc) {
    __shared__ uint32_t lds[5];
    if (sc->err) return;
    const int32_t l = sc->last_front;
    const int64_t R = sc->num_from_last;
    const int64_t ne = totals[0];
    const int64_t base = (int64_t)blockIdx.x * kOsTile;
    int64_t op = off[blockIdx.x], oq = off[nbp + blockIdx.x];
    for (int it = 0; it < kOsTile / 256; ++it) {
        const int64_t p = base + it * 256 + threadIdx.x;
        uint8_t f = 0;
        bool member = false;
        if (p < N) {
            f = selflag[p];
            member = rank[p] == l;
        }
        const uint32_t isP = f == 2 ? 1u : 0u;
        const uint32_t isQ = (member && f != 2) ? 1u : 0u;
        // picks in the low 16 bits, unpicked members in the high ones (<= 256 each)
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan(isP | (isQ << 16), lds, &tot);
        if (isP) selflag[p] = (R >= ne || op + (ex & 0xffffu) < R) ? 1 : 0;
        if (isQ) selflag[p] = (R > ne && oq + (ex >> 16) < R - ne) ? 1 : 0;
        op += tot & 0xffffu;
        oq += tot >> 16;
    }
}

size_t oneshot_temp_bytes(int64_t n) {
    const int64_t nb = (n + kOsTile - 1) / kOsTile;
    return (size_t)(2 * (nb + 64) + 64) * sizeof(uint32_t);
}

void run_compact(const uint8_t *flag, int64_t N, int32_t *out, int64_t K, uint32_t *temp,
                 DevScalars *sc, nsga3_info *info, hipStream_t s) {
    if (N <= kCompactOne) {
        hipLaunchKernelGGL(k_compact_one, dim3(1), dim3(1024), 0, s, flag, N, out, K, sc, info);
        return;
    }
    compact_flags(flag, N, out, K, temp, &sc->n_selected, s);
    if (info) hipLaunchKernelGGL(k_finalize, dim3(1), dim3(64), 0, s, info, K, sc);
}

int normalize_partial_blocks(int64_t N) {
    int64_t nb = (N + kNormThreads - 1) / kNormThreads;
    if (nb > kNormBlocksMax) nb = kNormBlocksMax;
    if (nb < 1) nb = 1;
    return (int)nb;
}

// Lanes that share a point of the association: few points leave the chip idle
// while each lane walks the references alone, many pay for every lane's own
// normalisation, and many references are worth more lanes.  1 / 4 / 16 lanes, us
// (M = 5): N = 3000, 100 references 14.6 / 8.2 / 7.0; 10000, 100 15.4 / 9.2 / 17.7, 500
// 50.0 / 20.7 / 16.3; 20000, 100 15.9 / 15.3 / 30.4, 500 50.0 / 22.8 / 27.0; 50000, 100 19.8
// / 28.1 / 68.3, 300 37.6 / 32.2 / 47.7; 100000, 500 59 / 63 / 81; 200000, 2000 236 / 275 / 370.
static int assoc_split(int64_t N, int H) {
    if (N <= 4096 || (N <= 16384 && H >= 512)) return 16;
    return N <= 32768 || (N <= 65536 && H >= 256) ? 4 : 1;
}

hipError_t run_select_stage(const SelectViews &v, hipStream_t s) {
    const int64_t N = v.N;
    const int M = v.M;
    const int nparts = normalize_partial_blocks(N);
    v.mark();
    switch (M) {
#define NSGA3_CASE(m)                                                                               \
    case m:                                                                                         \
        hipLaunchKernelGGL(k_extreme<m>, dim3(nparts), dim3(kNormThreads), 0, s, v.objs, N, v.rank, \
                           v.sc, v.p_asf, v.p_idx, v.p_nad);                                        \
        break;
        NSGA3_CASE(2) NSGA3_CASE(3) NSGA3_CASE(4) NSGA3_CASE(5) NSGA3_CASE(6) NSGA3_CASE(7)
        NSGA3_CASE(8) NSGA3_CASE(9) NSGA3_CASE(10) NSGA3_CASE(11) NSGA3_CASE(12) NSGA3_CASE(13)
        NSGA3_CASE(14) NSGA3_CASE(15) NSGA3_CASE(16)
#undef NSGA3_CASE
        default: return hipErrorInvalidValue;
    }
    const unsigned nbN = (unsigned)((N + 255) / 256);
    v.mark();
    const unsigned nbW = (unsigned)((N + 127) / 128);  // 32 points per wave, 4 waves per block
    const int S = assoc_split(N, v.H);
    const unsigned nbS = (unsigned)((N * S + kNormThreads - 1) / kNormThreads);
    switch (M) {
#define NSGA3_ASSOC(m, q)                                                                           \
    hipLaunchKernelGGL((k_associate<m, q>), dim3(nbS), dim3(kNormThreads), 0, s, v.objs, N, v.rank, \
                       v.rhat64, v.rhat32, v.H, v.niche, v.dist, v.dist64, v.rho, v.bcount,         \
                       v.selflag, v.sc)
#define NSGA3_CASE(m)                                                                               \
    case m:                                                                                         \
        if (v.assoc_mode == NSGA3_ASSOC_BF16)                                                       \
            hipLaunchKernelGGL(k_associate_bf16<m>, dim3(nbW), dim3(256), 0, s, v.objs, N, v.rank,  \
                               v.rhat64, v.rhat16, v.H, v.niche, v.dist, v.dist64, v.rho,           \
                               v.bcount, v.selflag, v.sc);                                          \
        else if (S == 16)                                                                           \
            NSGA3_ASSOC(m, 16);                                                                     \
        else if (S == 4)                                                                            \
            NSGA3_ASSOC(m, 4);                                                                      \
        else                                                                                        \
            NSGA3_ASSOC(m, 1);                                                                      \
        break;
        NSGA3_CASE(2) NSGA3_CASE(3) NSGA3_CASE(4) NSGA3_CASE(5) NSGA3_CASE(6) NSGA3_CASE(7)
        NSGA3_CASE(8) NSGA3_CASE(9) NSGA3_CASE(10) NSGA3_CASE(11) NSGA3_CASE(12) NSGA3_CASE(13)
        NSGA3_CASE(14) NSGA3_CASE(15) NSGA3_CASE(16)
#undef NSGA3_ASSOC
#undef NSGA3_CASE
        default: return hipErrorInvalidValue;
    }
    v.mark();
    if (N <= kNicheOne && v.H <= kNicheOneRefs && v.niching_mode != NSGA3_NICHING_ONESHOT) {
        hipLaunchKernelGGL(k_niche_one, dim3(1), dim3(1024), 0, s, (int)N, v.H, v.rank, v.niche,
                           v.dist64, v.rho, v.bcount, v.bstart, v.bcursor, v.gstart, v.selflag,
                           v.selected, v.K, v.sc, v.info);
        v.mark();
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_niche_plan, dim3(1), dim3(1024), 0, s, v.H, v.rho, v.bcount, v.bstart,
                       v.bcursor, v.gstart, v.sc);
    hipLaunchKernelGGL(k_bucket_scatter, dim3(nbN), dim3(256), 0, s, N, v.H, v.rank, v.niche, v.dist64,
                       v.bcursor, v.bd, v.bi, v.sc);
    if (v.niching_mode == NSGA3_NICHING_ONESHOT) {
        hipLaunchKernelGGL(k_oneshot_pick, dim3((unsigned)((v.H + 3) / 4)), dim3(256), 0, s, v.H,
                           v.rho, v.bstart, v.bd, v.bi, v.selflag, v.sc);
        const int64_t nbo = (N + kOsTile - 1) / kOsTile;
        const int64_t nbp = nbo + 64;
        uint32_t *cnt = v.temp, *totals = v.temp + 2 * nbp;
        hipLaunchKernelGGL(k_oneshot_count, dim3((unsigned)nbo), dim3(256), 0, s, N, v.rank,
                           v.selflag, cnt, nbp, v.sc);
        scan_inplace(cnt, nbo, totals, s);
        scan_inplace(cnt + nbp, nbo, totals + 1, s);
        hipLaunchKernelGGL(k_oneshot_apply, dim3((unsigned)nbo), dim3(256), 0, s, N, v.rank,
                           v.selflag, cnt, nbp, totals, v.sc);
    } else {
        // at most ceil(|F_l| / kRankMembers) + H groups, |F_l| <= N
        const unsigned nbG = (unsigned)((N + kRankMembers - 1) / kRankMembers + v.H);
        hipLaunchKernelGGL(k_bucket_rank, dim3(nbG), dim3(kRankGroup), 0, s, v.H, v.rho, v.bstart,
                           v.gstart, v.bd, v.bi, v.selflag, v.sc);
    }
    run_compact(v.selflag, N, v.selected, v.K, v.temp, v.sc, v.info, s);
    v.mark();
    return hipGetLastError();
}

hipError_t run_refs(const RefArgs &R, int M, DevScalars *sc, hipStream_t s) {
    hipLaunchKernelGGL(k_refs, dim3((unsigned)((R.Hpad + 255) / 256)), dim3(256), 0, s, R, M, sc);
    return hipGetLastError();
}

}  // namespace nsga3
