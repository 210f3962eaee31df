// Exact projection of points from given k nearest landmarks, FP64 throughout,
// for M-dimensional landmark positions (M = 2 or 3): G lanes (16, 32 or 64, the
// smallest that holds k) take a point, 64 / G points a wavefront.
//   1. lane q < k: the exact squared distance of neighbour q; the four lanes of a
//      quad read their four rows together, 64 consecutive bytes of each at a time;
//   2. the list sorted by (distance, index) when it is not already;
//   3. scores (rank-weighted mean and variance, exponential, cutoff);
//   4. the pairs with non-zero weight spread over the lanes, the segment
//      coordinate by polarisation, D = 1/2 + (delta_a^2 - delta_b^2) / (2 |L_a -
//      L_b|^2), with 1 / (2 |L_a - L_b|^2) from a g x g FP64 table when the caller
//      has one, else from the rows; a pair whose distances exceed 10^6 |L_a -
//      L_b|^2, where polarisation loses digits, is projected directly, D =
//      <x - L_a, H> / |H|^2;
//   5. sums over the lanes (DPP within 16), Cramer's rule, or the centroid of the
//      neighbours' positions for a degenerate neighbourhood or a numerically
//      singular system (det <= 1e-9 (tr/M)^M).
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "esom_internal.h"

namespace esom {

constexpr int LP_THREADS = 256;
constexpr double LP_POLAR_MAX = 1e6;  // delta^2 / |H|^2 beyond which a pair is projected directly

// One neighbour as the pair loop reads it (two 16-byte LDS reads).
struct __align__(16) LpNeighbour {
    double d2, s;
    float l[3];
    unsigned pos;
};

// LDS of a block: the neighbours of its groups, then the pairs as (a, b) bytes.
__host__ __device__ inline size_t lp_lds_bytes(int k) {
    return sizeof(LpNeighbour) * LP_THREADS + sizeof(unsigned short) * (size_t)(k * (k - 1) / 2);
}

template <int CTRL>
__device__ __forceinline__ double lp_dpp(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lp_quad_sum(double v) {
    v += lp_dpp<0xB1>(v);  // lanes 1 0 3 2
    v += lp_dpp<0x4E>(v);  // lanes 2 3 0 1
    return v;
}
// Sum over the G lanes of a group, the same on all of them.
template <int G>
__device__ __forceinline__ double lp_sum(double v) {
    v = lp_quad_sum(v);
    v += lp_dpp<0x141>(v);  // the other quad of 8 lanes (mirrored)
    v += lp_dpp<0x140>(v);  // the other half of 16 lanes (mirrored)
    if constexpr (G >= 32) v += __shfl_xor(v, 16);
    if constexpr (G >= 64) v += __shfl_xor(v, 32);
    return v;
}
// The group's bits of a wavefront's ballot.
template <int G>
__device__ __forceinline__ bool lp_any(bool b) {
    const unsigned long long m = __ballot(b);
    if constexpr (G == 64) return m != 0ull;
    return ((m >> ((threadIdx.x & 63) / G * G)) & ((1ull << (G & 63)) - 1ull)) != 0ull;
}
__device__ __forceinline__ void lp_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The block's pair list (a, b), a < b < kact, in row order.  Ends with a barrier.
__device__ __forceinline__ void lp_pairs(unsigned short *pairs, int kact) {
    for (int a = threadIdx.x; a < kact - 1; a += LP_THREADS)
        for (int b = a + 1, p = a * (2 * kact - a - 1) / 2; b < kact; ++b, ++p)
            pairs[p] = (unsigned short)(a | (b << 8));
    __syncthreads();
}

__device__ __forceinline__ double lp_det3(double a00, double a01, double a02, double a10, double a11, double a12,
                                          double a20, double a21, double a22) {
    return a00 * (a11 * a22 - a12 * a21) - a01 * (a10 * a22 - a12 * a20) + a02 * (a10 * a21 - a11 * a20);
}

// Values t0 .. t0 + N - 1 of a row of d floats (4-byte aligned), 0 past its end.
struct __attribute__((packed, aligned(4))) LpFloat4 {
    float x, y, z, w;
};
template <int N>
__device__ __forceinline__ void lp_load(const float *x, int t0, int d, float (&v)[N]) {
    if (t0 + N <= d) {
#pragma unroll
        for (int q = 0; q < N / 4; ++q) {
            const LpFloat4 f = *reinterpret_cast<const LpFloat4 *>(x + t0 + 4 * q);
            v[4 * q] = f.x;
            v[4 * q + 1] = f.y;
            v[4 * q + 2] = f.z;
            v[4 * q + 3] = f.w;
        }
    } else {
#pragma unroll
        for (int t = 0; t < N; ++t) v[t] = t0 + t < d ? x[t0 + t] : 0.f;
    }
}

// <x - L_u, H> and |H|^2 of the rows at positions u, v (H = L_v - L_u), U quads of
// dimensions loaded at a time: 4 where every pair comes here; 1 where the table
// serves almost all of them and the registers are the other waves' (with 4 the
// 3-D projection of 200k points took 218 us for 177).
template <int U>
__device__ __forceinline__ void lp_direct(const ListArgs &e, const float *x, unsigned u, unsigned v, double &xH,
                                          double &HH) {
    const float4 *Lu = reinterpret_cast<const float4 *>(e.Lpad + (size_t)u * e.dp);
    const float4 *Lv = reinterpret_cast<const float4 *>(e.Lpad + (size_t)v * e.dp);
    xH = HH = 0.0;
    for (int c = 0; c < e.dp / (4 * U); ++c) {
        float4 lu[U], lv[U];
        float xv[4 * U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            lu[q] = Lu[U * c + q];
            lv[q] = Lv[U * c + q];
        }
        lp_load<4 * U>(x, 4 * U * c, e.d, xv);
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const float a[4] = {lu[q].x, lu[q].y, lu[q].z, lu[q].w}, b[4] = {lv[q].x, lv[q].y, lv[q].z, lv[q].w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double H = (double)b[t] - (double)a[t];
                HH = fma(H, H, HH);
                xH = fma((double)xv[4 * q + t] - (double)a[t], H, xH);  // H is 0 past d
            }
        }
    }
}

// One point per group of G lanes: pi the point, on = the group has one.  All
// lanes of the wavefront call it together.  Writes the output, and (e.out_idx /
// e.out_d2) the sorted list.
template <int G, int M>
__device__ __forceinline__ void lp_point(const ListArgs &e, int64_t pi, bool on, LpNeighbour *nb,
                                         const unsigned short *pairs) {
    const int lane = threadIdx.x & (G - 1);
    const int k = e.k, kact = e.use_cutoff ? k - 1 : k;
    const float *x = e.X + (on ? pi : 0) * e.ldx;
    const bool act = on && lane < k;
    int jq = act ? e.knn_idx[pi * k + lane] : 0;
    const bool bad1 = act && (jq < 0 || jq >= e.g);
    if (bad1) jq = 0;
    const bool bad = lp_any<G>(bad1);
    // exact squared distances, by quads
    const unsigned pos = (unsigned)e.ipos[jq];
    double dq = 0.0;
    {
        const float4 *rows[4];
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        const int qb = (threadIdx.x & 63) & ~3;
#pragma unroll
        for (int s = 0; s < 4; ++s)
            rows[s] = reinterpret_cast<const float4 *>(e.Lpad + (size_t)__shfl(pos, qb + s) * e.dp) + (lane & 3);
        for (int c = 0; c < e.dp / 16; ++c) {
            float4 lv[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) lv[s] = rows[s][4 * c];
            const int t0 = 16 * c + 4 * (lane & 3);
            double xv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) xv[t] = t0 + t < e.d ? (double)x[t0 + t] : 0.0;  // the rows are 0 there
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double d0 = xv[0] - (double)lv[s].x, d1 = xv[1] - (double)lv[s].y;
                const double d2 = xv[2] - (double)lv[s].z, d3 = xv[3] - (double)lv[s].w;
                acc[s] = fma(d0, d0, acc[s]);
                acc[s] = fma(d1, d1, acc[s]);
                acc[s] = fma(d2, d2, acc[s]);
                acc[s] = fma(d3, d3, acc[s]);
            }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double t = lp_quad_sum(acc[s]);
            dq = (lane & 3) == s ? t : dq;
        }
    }
    // Sorted by (distance, index).  A point without a list (its entries all stand for
    // landmark 0) or with NaN distances shares the wavefront with points to sort, so the
    // ranks are a permutation of the places for it too: such a list keeps its places,
    // and NaN ranks as +inf.  (A place that no entry took would hold other data, and its
    // index is used for loads.)
    const double dprev = __shfl_up(dq, 1);
    const int jprev = __shfl_up(jq, 1);
    int rank = lane;
    if (__ballot(act && lane > 0 && (dprev > dq || (dprev == dq && jprev > jq))) != 0ull) {
        rank = 0;
        const double dr = bad ? (double)lane : dq == dq ? dq : (double)INFINITY;
        const int gb = (threadIdx.x & 63) & ~(G - 1);
        for (int p = 0; p < k; ++p) {
            const double dp = __shfl(dr, gb + p);
            const int jp = __shfl(jq, gb + p);
            rank += (dp < dr || (dp == dr && jp < jq)) ? 1 : 0;
        }
        if (lane >= k) rank = lane;
    }
    nb[rank].d2 = dq;
    nb[rank].pos = pos;
    reinterpret_cast<int *>(nb[rank].l)[0] = jq;
    lp_fence();
    const double d2r = act ? nb[lane].d2 : 0.0;
    const int jr = act ? reinterpret_cast<const int *>(nb[lane].l)[0] : 0;
    if (act && !bad) {
        if (e.out_idx) e.out_idx[pi * k + lane] = jr;
        if (e.out_d2) e.out_d2[pi * k + lane] = (float)d2r;
    }
    // scores
    const double dl = sqrt(d2r);
    const double w = act ? 1.0 / (double)(lane + 1) : 0.0;
    const double mu = lp_sum<G>(w * dl) / e.Wk;
    const double dev = act ? dl - mu : 0.0;
    const double var = lp_sum<G>(w * dev * dev) / e.Wk;
    const double d0 = sqrt(nb[0].d2), dk = sqrt(nb[k - 1].d2);
    const bool degenerate = d0 == dk;
    double s = 0.0;
    if (act && !degenerate) {
        const double ex = var > 1e-30 * mu * mu ? exp(e.boost * (mu - dl) / sqrt(var)) : 1.0;
        const double c = e.use_cutoff ? 1.0 - exp(e.cutoff * (dl / dk - 1.0)) : 1.0;
        s = ex * c;
    }
    double lr[M];
#pragma unroll
    for (int c = 0; c < M; ++c) lr[c] = act ? (double)e.l[(size_t)M * jr + c] : 0.0;
    lp_fence();
    nb[lane].s = s;
#pragma unroll
    for (int c = 0; c < M; ++c) nb[lane].l[c] = (float)lr[c];
    lp_fence();
    // gravity, then the pairs: m = the upper triangle of M row by row
    constexpr int NM = M * (M + 1) / 2;
    double m[NM], r[M];
    const double gs = e.gravity * s;
    for (int c = 0, i = 0; c < M; ++c) {
        r[c] = gs * lr[c];
        for (int c2 = c; c2 < M; ++c2, ++i) m[i] = c2 == c ? gs : 0.0;
    }
    const int np = degenerate || bad || !on ? 0 : kact * (kact - 1) / 2;
    for (int p = lane; p < np; p += G) {
        const unsigned ab = pairs[p];
        const LpNeighbour A = nb[ab & 255], B = nb[ab >> 8];
        double inv;  // 1 / (2 |H|^2), 0 for coincident landmarks
        double xH = 0.0, HH = 0.0;
        if (e.tab) {
            inv = e.tab[(size_t)A.pos * e.g + B.pos];
        } else {
            lp_direct<M == 2 ? 4 : 1>(e, x, A.pos, B.pos, xH, HH);
            inv = HH > 0.0 ? 0.5 / HH : 0.0;
        }
        if (!(inv > 0.0)) continue;
        double D = fma(A.d2 - B.d2, inv, 0.5);
        if (!e.tab) {
            D = xH / HH;
        } else if (2.0 * B.d2 * inv > LP_POLAR_MAX) {  // delta^2 ascends: B's is the larger
            lp_direct<M == 2 ? 4 : 1>(e, x, A.pos, B.pos, xH, HH);
            D = xH / HH;
        }
        double h[M], hh = 0.0, hl = 0.0;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            h[c] = (double)B.l[c] - (double)A.l[c];
            hh = fma(h[c], h[c], hh);
            hl = fma(h[c], (double)A.l[c], hl);
        }
        if (hh == 0.0) continue;  // coincident positions
        const double ih = 1.0 / hh;
        const double q = A.s * B.s * (e.adjust == 1.0 ? ih : pow(hh, -e.adjust));
        const double rhs = D + hl * ih, qh = q * ih;
        for (int c = 0, i = 0; c < M; ++c) {
            r[c] = fma(q * h[c], rhs, r[c]);
            for (int c2 = c; c2 < M; ++c2, ++i) m[i] = fma(qh * h[c], h[c2], m[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < NM; ++i) m[i] = lp_sum<G>(m[i]);
#pragma unroll
    for (int c = 0; c < M; ++c) r[c] = lp_sum<G>(r[c]);
    const double ssum = lp_sum<G>(s);
    double det, tr, lim;
    if constexpr (M == 2) {
        det = m[0] * m[2] - m[1] * m[1];
        tr = 0.5 * (m[0] + m[2]);
        lim = 1e-9 * tr * tr;
    } else {
        det = lp_det3(m[0], m[1], m[2], m[1], m[3], m[4], m[2], m[4], m[5]);
        tr = (m[0] + m[3] + m[5]) / 3.0;
        lim = 1e-9 * tr * tr * tr;
    }
    const bool centroid = degenerate || !(ssum > 0.0) || !(det > lim);
    double o[M];
    if (__ballot(on && !bad && centroid) != 0ull) {
#pragma unroll
        for (int c = 0; c < M; ++c) o[c] = lp_sum<G>(lr[c]) / k;
    }
    if (!centroid) {
        if constexpr (M == 2) {
            o[0] = (r[0] * m[2] - m[1] * r[1]) / det;
            o[1] = (m[0] * r[1] - m[1] * r[0]) / det;
        } else {
            o[0] = lp_det3(r[0], m[1], m[2], r[1], m[3], m[4], r[2], m[4], m[5]) / det;
            o[1] = lp_det3(m[0], r[0], m[2], m[1], r[1], m[4], m[2], r[2], m[5]) / det;
            o[2] = lp_det3(m[0], m[1], r[0], m[1], m[3], r[1], m[2], m[4], r[2]) / det;
        }
    }
    if (on && lane == 0) {
#pragma unroll
        for (int c = 0; c < M; ++c) e.out[(size_t)M * pi + c] = bad ? NAN : (float)o[c];
    }
    lp_fence();
}

}  // namespace esom
