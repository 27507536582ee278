// Per-point and per-instance arithmetic of the selection stages (internal),
// shared by the single-selection kernels and the batched engine so that both
// produce bit-identical results.
#pragma once

#include <float.h>

#include "common.h"

namespace nsga3 {

// a4: achievement scalarising function of one translated point g (Alg. S.5,
// weights 1 on axis j and 1e-6 elsewhere, applied as x 1e6) for every axis j,
// folded into running minima (lowest index on ties) and the nadir maxima.
template <int MM>
__device__ __forceinline__ void asf_fold(const double (&g)[MM], int M, int32_t i, double (&best)[MM],
                                         int32_t (&bidx)[MM], double (&nad)[MM]) {
#pragma unroll
    for (int k = 0; k < MM; ++k)
        if (k < M && g[k] > nad[k]) nad[k] = g[k];
    // the largest weighted value and the largest of the others, so that axis j's
    // maximum over the other axes is one of the two
    double m1 = -DBL_MAX, m2 = -DBL_MAX;
    int at = -1;
#pragma unroll
    for (int k = 0; k < MM; ++k) {
        if (k < M) {
            const double v = g[k] * 1e6;
            if (v > m1) { m2 = m1; m1 = v; at = k; }
            else if (v > m2) { m2 = v; }
        }
    }
#pragma unroll
    for (int j = 0; j < MM; ++j) {
        if (j < M) {
            double asf = j == at ? m2 : m1;
            if (g[j] > asf) asf = g[j];
            if (asf < best[j]) { best[j] = asf; bidx[j] = i; }
        }
    }
}

__device__ __forceinline__ double lane_read(double x, int l) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// a5: intercepts from the extreme points, by one whole wave (lane r holds
// row r of E; lanes >= M take part in nothing).  e[j] is the index
// of the extreme point of axis j, nadir[k] the largest translated value over
// S, z the ideal point.  Solves E b = 1 by Gaussian elimination with partial
// pivoting (largest |pivot|, lowest row on ties; singular when a pivot is
// <= 1e-10 max|E|); a = 1/b when every b_k is finite and positive and every
// 1/b_k finite, else the nadir; an intercept of exactly 0 becomes 1.  Every
// lane returns the same a and fallback code (0 hyperplane, 1 nadir, 2 unit
// guard).  Each entry goes through the same operations, in the same order, as
// in the one-row-at-a-time textbook elimination.
template <int M>
__device__ __forceinline__ int solve_intercepts_wave(const float *objs, const int32_t *e,
                                                     const double *nadir, const double (&z)[M],
                                                     double (&a)[M]) {
    const int lane = (int)lane_id();
    const bool own = lane < M;
    const int64_t er = e[own ? lane : 0];
    double row[M];
    double rhs = 1.0;
    double mx = 0.0;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        row[k] = (double)objs[er * M + k] - z[k];
        const double av = fabs(row[k]);
        mx = av > mx ? av : mx;
    }
    // (values of one lane come over by lane reads, M of them in less time than
    // the six exchanges of a reduction over the wave)
    double maxabs = 0.0;
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const double t = lane_read(mx, r);
        maxabs = t > maxabs ? t : maxabs;
    }
    bool ok = maxabs > 0.0;
#pragma unroll
    for (int c = 0; c < M; ++c) {
        const double av = fabs(row[c]);
        double pv = lane_read(av, c);
        int p = c;
#pragma unroll
        for (int r = c + 1; r < M; ++r) {
            const double v = lane_read(av, r);
            if (v > pv) { pv = v; p = r; }
        }
        p = __builtin_amdgcn_readfirstlane(p);
        ok = ok && pv > 1e-10 * maxabs;
        // rows c and p trade places
        double prow[M];
#pragma unroll
        for (int k = c; k < M; ++k) {
            const double rc = lane_read(row[k], c);
            prow[k] = lane_read(row[k], p);
            row[k] = lane == c ? prow[k] : (lane == p ? rc : row[k]);
        }
        const double hc = lane_read(rhs, c), prhs = lane_read(rhs, p);
        rhs = lane == c ? prhs : (lane == p ? hc : rhs);
        if (own && lane > c) {
            const double f = row[c] / prow[c];
#pragma unroll
            for (int k = c + 1; k < M; ++k) row[k] = row[k] - f * prow[k];
            row[c] = 0.0;
            rhs = rhs - f * prhs;
        }
    }
    if (ok) {
        double b[M];
#pragma unroll
        for (int c = M - 1; c >= 0; --c) {
            double s = lane_read(rhs, c);
#pragma unroll
            for (int k = c + 1; k < M; ++k) s = s - lane_read(row[k], c) * b[k];
            b[c] = s / lane_read(row[c], c);
        }
#pragma unroll
        for (int k = 0; k < M; ++k) {
            if (!(ok && __builtin_isfinite(b[k]) && b[k] > 0.0)) { ok = false; continue; }
            const double ak = 1.0 / b[k];
            if (!__builtin_isfinite(ak)) ok = false;
            a[k] = ak;
        }
    }
    int fb = 0;
    if (!ok) {
        fb = 1;
#pragma unroll
        for (int k = 0; k < M; ++k) a[k] = nadir[k];
    }
#pragma unroll
    for (int k = 0; k < M; ++k)
        if (a[k] == 0.0) { a[k] = 1.0; fb = 2; }
    return fb;
}

// a6: normalised point f' = (f - z) / a and its screening vector y = f' / max f'
// (the scale of y does not move the argmax of y . rhat).  Returns ||y||_1.
template <int M>
__device__ __forceinline__ float normalise_point(const float *f, const double *z, const double *a,
                                                 double (&fp)[M], float (&y)[M]) {
    double mx = 0.0;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        fp[k] = ((double)f[k] - z[k]) / a[k];
        mx = fp[k] > mx ? fp[k] : mx;
    }
    float l1 = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        y[k] = mx > 0.0 ? (float)(fp[k] / mx) : 0.0f;
        l1 += y[k];
    }
    return l1;
}

// Float64 residual distance of f' to the line of unit reference rd (Eq. (10)
// in its residual form ||f' - (f'.r) r||).
template <int M>
__device__ __forceinline__ double line_distance(const double (&fp)[M], const double *rd) {
    double s64 = 0.0;
#pragma unroll
    for (int k = 0; k < M; ++k) s64 = s64 + fp[k] * rd[k];
    double q = 0.0;
#pragma unroll
    for (int k = 0; k < M; ++k) {
        const double e = fp[k] - s64 * rd[k];
        q = q + e * e;
    }
    return sqrt(q);
}

// Float32 screening band: |s32 - s| <= (M + 3) u ||y||_2 <= (M + 3) u ||y||_1
// with u = 2^-24; a 4x margin keeps every reference within float64 reach of
// the best one.
template <int M>
__device__ __forceinline__ float fp32_band(float l1) {
    return 4.0f * (float)(M + 4) * 5.9604645e-8f * l1 + 1e-30f;
}

// a6 for one point: screen every reference with s = y . rhat in float32 (R is
// the H x M float32 unit references), re-score the survivors in float64.
// best = lowest index among the smallest distances; d1 <= d2 the two smallest.
// References go four at a time (independent chains; each s is summed in the
// same order as a one-at-a-time loop, and survivors are visited in ascending
// index order, so results do not depend on the grouping).
template <int M>
__device__ __forceinline__ float screen_dot(const float (&y)[M], const float *__restrict__ r) {
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < M; ++k) s = __fmaf_rn(y[k], r[k], s);
    return s;
}

template <int M>
__device__ __forceinline__ void associate_point(const double (&fp)[M], const float (&y)[M], float l1,
                                                const float *__restrict__ R,
                                                const double *__restrict__ rhat64, int H,
                                                int32_t &best, double &d1, double &d2) {
    float smax = -FLT_MAX;
    int j = 0;
    for (; j + 4 <= H; j += 4) {
        const float s0 = screen_dot<M>(y, R + (j + 0) * M), s1 = screen_dot<M>(y, R + (j + 1) * M);
        const float s2 = screen_dot<M>(y, R + (j + 2) * M), s3 = screen_dot<M>(y, R + (j + 3) * M);
        smax = fmaxf(smax, fmaxf(fmaxf(s0, s1), fmaxf(s2, s3)));
    }
    for (; j < H; ++j) smax = fmaxf(smax, screen_dot<M>(y, R + j * M));
    const float thr = smax - fp32_band<M>(l1);
    d1 = DBL_MAX;
    d2 = DBL_MAX;
    best = 0;
    auto consider = [&](int jj, float s) {
        if (s < thr) return;
        const double d = line_distance<M>(fp, rhat64 + (int64_t)jj * M);
        if (d < d1) { d2 = d1; d1 = d; best = jj; }
        else if (d < d2) { d2 = d; }
    };
    j = 0;
    for (; j + 4 <= H; j += 4) {
        const float s0 = screen_dot<M>(y, R + (j + 0) * M), s1 = screen_dot<M>(y, R + (j + 1) * M);
        const float s2 = screen_dot<M>(y, R + (j + 2) * M), s3 = screen_dot<M>(y, R + (j + 3) * M);
        consider(j, s0);
        consider(j + 1, s1);
        consider(j + 2, s2);
        consider(j + 3, s3);
    }
    for (; j < H; ++j) consider(j, screen_dot<M>(y, R + j * M));
}

// Near-tie rule: the two smallest distances differ by less than 1e-6 relative.
__device__ __forceinline__ bool near_tie(double d1, double d2) {
    return d2 != DBL_MAX && (d2 - d1) < 1e-6 * fmax(d2, 1e-300);
}

// a7 niche counts of one work-group.  cls = 0 counts reference `best` into
// rho, cls = 1 into bcount, cls < 0 counts nothing.  For H <= kLdsNicheRefs the
// work-group first tallies in LDS (hist: 2 * kLdsNicheRefs ints) and then adds
// each non-zero tally with one global atomic, so a popular reference takes one
// atomic per work-group instead of one per point.  Every thread of the
// work-group calls it; it ends with a barrier.
constexpr int kLdsNicheRefs = 2048;

__device__ __forceinline__ void niche_count_block(int H, int cls, int32_t best, int32_t *rho,
                                                  int32_t *bcount, int32_t *hist) {
    if (H <= kLdsNicheRefs) {
        for (int q = threadIdx.x; q < 2 * H; q += blockDim.x) hist[q] = 0;
        __syncthreads();
        if (cls >= 0) atomicAdd(&hist[cls * H + best], 1);
        __syncthreads();
        for (int q = threadIdx.x; q < 2 * H; q += blockDim.x) {
            const int32_t v = hist[q];
            if (v) atomicAdd(q < H ? &rho[q] : &bcount[q - H], v);
        }
        __syncthreads();
    } else if (cls >= 0) {
        atomicAdd(cls ? &bcount[best] : &rho[best], 1);
    }
}

// a8 bucket slot of one work-group's last-front members (member: this thread
// holds one, in bucket b).  With H <= kLdsNicheRefs each bucket's cursor takes
// one atomic per work-group (cnt: kLdsNicheRefs ints of LDS).  Every thread of
// the work-group calls it; it ends with a barrier.  Slots inside a bucket are
// in no particular order.
__device__ __forceinline__ int32_t bucket_slot_block(int H, bool member, int32_t b,
                                                     int32_t *bcursor, int32_t *cnt) {
    if (H > kLdsNicheRefs) return member ? atomicAdd(&bcursor[b], 1) : -1;
    for (int q = threadIdx.x; q < H; q += blockDim.x) cnt[q] = 0;
    __syncthreads();
    const int32_t local = member ? atomicAdd(&cnt[b], 1) : 0;
    __syncthreads();
    for (int q = threadIdx.x; q < H; q += blockDim.x) {
        const int32_t v = cnt[q];
        if (v) cnt[q] = atomicAdd(&bcursor[q], v);
    }
    __syncthreads();
    const int32_t slot = member ? cnt[b] + local : -1;
    __syncthreads();
    return slot;
}

// Unit reference j (float64, float32); false when the row is invalid
// (non-finite, negative entry, zero norm).
__device__ __forceinline__ bool unit_reference(const float *refs, int j, int M, double *r64,
                                               float *r32) {
    double nn = 0.0;
    bool bad = false;
    for (int k = 0; k < M; ++k) {
        const float f = refs[(int64_t)j * M + k];
        bad |= !__builtin_isfinite(f) || f < 0.0f;
        const double v = (double)f;
        nn = nn + v * v;
    }
    const double n = sqrt(nn);
    bad |= !(n > 0.0) || !__builtin_isfinite(n);
    if (bad) return false;
    for (int k = 0; k < M; ++k) {
        const double r = (double)refs[(int64_t)j * M + k] / n;
        r64[(int64_t)j * M + k] = r;
        r32[(int64_t)j * M + k] = (float)r;
    }
    return true;
}

__device__ __forceinline__ uint16_t bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);  // finite inputs only
}

// Unit reference directions in float64 and float32, and in bfloat16 for the
// matrix-core screening: [Hpad x KP] (KP = 8 for M <= 8, else 16), rows and
// columns beyond (H, M) zero.
struct RefArgs {
    const float *refs;
    int H, Hpad, KP;
    double *rhat64;
    float *rhat32;
    uint16_t *rhat16;
};

__device__ __forceinline__ void reference_item(const RefArgs &R, int M, int j, DevScalars *sc) {
    if (j < R.Hpad && R.rhat16) {
        for (int k = 0; k < R.KP; ++k) R.rhat16[(int64_t)j * R.KP + k] = 0;
    }
    if (j >= R.H) return;
    if (!unit_reference(R.refs, j, M, R.rhat64, R.rhat32)) {
        atomicOr(&sc->err, (uint32_t)kErrBadRef);
        return;
    }
    if (R.rhat16)
        for (int k = 0; k < M; ++k)
            R.rhat16[(int64_t)j * R.KP + k] = bf16_rne(R.rhat32[(int64_t)j * M + k]);
}

// Per-call scalars, by one work-group of at least 16 threads.
__device__ __forceinline__ void init_scalars(DevScalars *sc, int t) {
    if (t == 0) {
        sc->err = 0;
        sc->last_front = 0;
        sc->num_fronts = 0;
        sc->last_front_size = 0;
        sc->n_before = 0;
        sc->num_from_last = 0;
        sc->fallback = 0;
        sc->near_ties = 0;
        sc->nf = sc->nu = 0;
        sc->bar_count = 0;
        sc->bar_gen = 0;
        sc->level_V = 0;
        sc->ref_thr = 0;
        sc->ext_done = 0;
    }
    if (t < 16) {
        sc->min_key[t] = 0xffffffffu;
        sc->a[t] = 1.0;
        sc->z[t] = 0.0;
    }
}

}  // namespace nsga3
