// Online SOM training support and the fit of added landmarks (supervised
// training of self-organizing maps: the user's 2-D map is the topology, new
// landmarks get high-dimensional positions fitted from their 2-D neighbours).
//
// A training step on a large batch gathers its points into a contiguous buffer,
// finds each point's best-matching landmark with the exact nearest-landmark
// path, and applies the averaged online update (esom_update.hip, kind 2); small
// batches take a direct path of two kernels.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "esom_internal.h"

namespace esom {

// Wavefront minima (device library, DPP reductions).
extern "C" __device__ double __ockl_wfred_min_f64(double);
extern "C" __device__ int __ockl_wfred_min_i32(int);

constexpr int SOM_WAVES = 4;             // wavefronts per block
constexpr int SOM_BLEND_J = 2;           // landmarks per blend block
constexpr int SOM_DIRECT_BATCH = 4096;   // largest batch of the direct path
constexpr int SOM_DIRECT_G = 4096;       // most landmarks of the direct path

// Xb[i] = X[rows[i]] (zeros for rows outside [0, n)); one thread per element.
__global__ void som_gather(const float *__restrict__ X, int64_t n, int64_t ldx, int d,
                           const int32_t *__restrict__ rows, int B, float *__restrict__ Xb) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)B * d) return;
    const int i = (int)(e / d), c = (int)(e % d);
    const int32_t r = rows[i];
    Xb[e] = (r >= 0 && r < n) ? X[(int64_t)r * ldx + c] : 0.f;
}

// nearest[i] = -1 where rows[i] is outside [0, n): that entry presents no point.
__global__ void som_mask(const int32_t *__restrict__ rows, int B, int64_t n, int32_t *__restrict__ nearest) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < B && (rows[i] < 0 || rows[i] >= n)) nearest[i] = -1;
}

hipError_t launch_som_gather(const float *X, int64_t n, int64_t ldx, int d, const int32_t *rows, int B,
                             float *Xb, hipStream_t s) {
    const int64_t tot = (int64_t)B * d;
    hipLaunchKernelGGL(som_gather, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, X, n, ldx, d, rows,
                       B, Xb);
    return hipGetLastError();
}

hipError_t launch_som_mask(const int32_t *rows, int B, int64_t n, int32_t *nearest, hipStream_t s) {
    hipLaunchKernelGGL(som_mask, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, rows, B, n, nearest);
    return hipGetLastError();
}

// ---------------------------------------------------------------- small batches
// A training step on a batch of at most SOM_DIRECT_BATCH points takes two
// launches and no scratch besides the list of nearest landmarks:
//   som_bmu    the batch points' nearest landmarks by FP64 distances to all g
//              landmarks (ties to the lower index);
//   som_blend  L_j += (alpha / batch) sum_i h(j, b_i) (x_i - L_j) straight from
//              the batch's rows.
// The general path (gather, landmark preparation, MFMA screen, exact path, mask,
// sums, blend: ten or eleven launches) is for larger batches: its screen costs less
// per point, but its launches and the preparation take most of the 69 us of a step of
// 5000 points (400 landmarks, 32-D).  Batch 1024: 397 us a step by that path as it
// was, with a counting sort and a blend that formed its weights per dimension, now
// 30 us.

// One wavefront per PW points; the block's wavefronts share landmark tiles of
// 64 TR rows in LDS (odd row stride: no bank conflicts), lane = TR landmarks.
// Bound by the latency of the tile loads, hence TR = 4 and 32 loads of a thread
// in flight where that tile leaves room for two blocks per CU (d <= 64).  The
// batch's rows are gathered straight from X.  nearest[i] = -1 for an entry
// outside [0, n) and for a NaN point.
template <int PW, int TR>
__global__ void __launch_bounds__(64 * SOM_WAVES) som_bmu(const float *__restrict__ X, int64_t n, int64_t ldx, int d,
                                                          const float *__restrict__ L, int g,
                                                          const int32_t *__restrict__ rows, int B,
                                                          int32_t *__restrict__ nearest) {
    extern __shared__ __align__(16) unsigned char bsm[];
    double *xs = reinterpret_cast<double *>(bsm);                              // SOM_WAVES x PW x d
    float *tile = reinterpret_cast<float *>(xs + (size_t)SOM_WAVES * PW * d);  // 64 TR rows
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i0 = (blockIdx.x * SOM_WAVES + wv) * PW;
    double *xw = xs + (size_t)wv * PW * d;
    unsigned live = 0u;  // bit p: entry i0 + p presents a point
#pragma unroll
    for (int p = 0; p < PW; ++p) {
        const int32_t r = i0 + p < B ? rows[i0 + p] : -1;
        const bool ok = r >= 0 && r < n;
        live |= (ok ? 1u : 0u) << p;
        const float *xr = X + (ok ? (int64_t)r * ldx : 0);
        for (int t = lane; t < d; t += 64) xw[p * d + t] = ok ? (double)xr[t] : 0.0;
    }
    double best[PW];
    int bj[PW];
#pragma unroll
    for (int p = 0; p < PW; ++p) {
        best[p] = INFINITY;
        bj[p] = 0x7fffffff;
    }
    const int rs = d | 1;
    constexpr int NT = 64 * SOM_WAVES, LD = 32;  // loads of a thread in flight
    const int step_r = NT / d, step_t = NT % d;
    for (int v0 = 0; v0 < g; v0 += 64 * TR) {
        __syncthreads();
        // the tile's rows are contiguous in L
        const int cnt = (g - v0 < 64 * TR ? g - v0 : 64 * TR) * d;
        const float *Lt = L + (size_t)v0 * d;
        int r = (int)threadIdx.x / d, t = (int)threadIdx.x % d;
        for (int e0 = threadIdx.x; e0 < cnt; e0 += LD * NT) {
            float x[LD];
#pragma unroll
            for (int i = 0; i < LD; ++i) x[i] = e0 + i * NT < cnt ? Lt[e0 + i * NT] : 0.f;
#pragma unroll
            for (int i = 0; i < LD; ++i) {
                if (e0 + i * NT < cnt) tile[r * rs + t] = x[i];
                r += step_r;
                t += step_t;
                if (t >= d) {
                    t -= d;
                    ++r;
                }
            }
        }
        __syncthreads();
        const float *Lv[TR];
        double s[TR][PW];
#pragma unroll
        for (int k = 0; k < TR; ++k) {
            Lv[k] = tile + (v0 + 64 * k + lane < g ? 64 * k + lane : 0) * rs;
#pragma unroll
            for (int p = 0; p < PW; ++p) s[k][p] = 0.0;
        }
#pragma unroll 8
        for (int q = 0; q < d; ++q) {
            double lv[TR];
#pragma unroll
            for (int k = 0; k < TR; ++k) lv[k] = (double)Lv[k][q];
#pragma unroll
            for (int p = 0; p < PW; ++p) {
                const double xq = xw[p * d + q];
#pragma unroll
                for (int k = 0; k < TR; ++k) {
                    const double df = xq - lv[k];
                    s[k][p] = fma(df, df, s[k][p]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < TR; ++k)
#pragma unroll
            for (int p = 0; p < PW; ++p)
                if (v0 + 64 * k + lane < g && s[k][p] < best[p]) {  // ascending per lane: the lower index wins a tie
                    best[p] = s[k][p];
                    bj[p] = v0 + 64 * k + lane;
                }
    }
#pragma unroll
    for (int p = 0; p < PW; ++p) {
        const double m = __ockl_wfred_min_f64(best[p]);
        int j = __ockl_wfred_min_i32(best[p] == m ? bj[p] : 0x7fffffff);
        if (m == INFINITY) {
            // no finite distance: the infinite ones compete by index
            int jf = 0x7fffffff;
            for (int v = lane; v < g && jf == 0x7fffffff; v += 64) {
                double s = 0.0;
                for (int q = 0; q < d; ++q) {
                    const double df = xw[p * d + q] - (double)L[(size_t)v * d + q];
                    s = fma(df, df, s);
                }
                if (s == INFINITY) jf = v;
            }
            j = __ockl_wfred_min_i32(jf);
        }
        if (lane == 0 && i0 + p < B) nearest[i0 + p] = ((live >> p) & 1u) && j < g ? j : -1;
    }
}

// A block of NW wavefronts takes SOM_BLEND_J landmarks j: their weights h(j, b)
// for every landmark b and the batch's (row, nearest) pairs go to LDS, then each
// wavefront adds its share of the batch's rows, LP lanes per row over the
// dimensions, and all partial sums meet in LDS.  Bound by the latency of the
// gathered rows, so many are in flight: at batch 1024, 32-D, 4 wavefronts with 8
// rows each took 93 us, 16 wavefronts 27 us, and two rows per wavefront load
// and 16 loads in flight (2 rounds) 17 us.
template <int LP, int NQ, int NW>
__global__ void __launch_bounds__(64 * NW) som_blend(const float *__restrict__ X, int64_t ldx, int d,
                                                     float *__restrict__ L, const float *__restrict__ l2d, int g,
                                                     const int32_t *__restrict__ rows,
                                                     const int32_t *__restrict__ nearest, int B, float sigma,
                                                     float alpha, const uint8_t *__restrict__ frozen) {
    extern __shared__ __align__(16) unsigned char ssm[];
    double *hs = reinterpret_cast<double *>(ssm);                     // SOM_BLEND_J x g
    int2 *pts = reinterpret_cast<int2 *>(hs + (size_t)SOM_BLEND_J * g);  // B: (row, nearest)
    constexpr int PP = 64 / LP, NG = NW * PP;  // rows per wavefront load, groups of lanes in the block
    __shared__ double red[NG][SOM_BLEND_J][LP * NQ];
    __shared__ double rden[NG][SOM_BLEND_J];
    const int lane = threadIdx.x % LP, gr = threadIdx.x / LP;
    const int j0 = blockIdx.x * SOM_BLEND_J;
    const double s2 = 2.0 * (double)sigma * (double)sigma;
    for (int p = threadIdx.x; p < B; p += blockDim.x) {
        const int b = nearest[p];
        pts[p] = make_int2(b >= 0 ? rows[p] : 0, b);
    }
    for (int e = threadIdx.x; e < SOM_BLEND_J * g; e += blockDim.x) {
        const int i = e / g, b = e % g, j = min(j0 + i, g - 1);
        double w;
        if (sigma == 0.f) {
            w = b == j ? 1.0 : 0.0;
        } else {
            const double dx = (double)l2d[2 * j] - (double)l2d[2 * b], dy = (double)l2d[2 * j + 1] - (double)l2d[2 * b + 1];
            w = exp(-(dx * dx + dy * dy) / s2);
        }
        hs[e] = w;
    }
    __syncthreads();
    double acc[SOM_BLEND_J][NQ], den[SOM_BLEND_J];
#pragma unroll
    for (int i = 0; i < SOM_BLEND_J; ++i) {
        den[i] = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[i][q] = 0.0;
    }
    constexpr int U = 16 / NQ;  // rows in flight per group
    for (int p0 = gr; p0 < B; p0 += NG * U) {
        int b[U];
        float x[U][NQ];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int at = p0 + u * NG;
            const int2 pt = pts[at < B ? at : p0];
            b[u] = at < B ? pt.y : -1;
            const float *xr = X + (int64_t)pt.x * ldx;
#pragma unroll
            for (int q = 0; q < NQ; ++q) x[u][q] = b[u] >= 0 && lane + LP * q < d ? xr[lane + LP * q] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < SOM_BLEND_J; ++i) {
                // an entry that presents no point: weight and row are 0
                const double w = b[u] >= 0 ? hs[i * g + b[u]] : 0.0;
                den[i] += w;
#pragma unroll
                for (int q = 0; q < NQ; ++q) acc[i][q] = fma(w, (double)x[u][q], acc[i][q]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < SOM_BLEND_J; ++i) {
        if (lane == 0) rden[gr][i] = den[i];
#pragma unroll
        for (int q = 0; q < NQ; ++q) red[gr][i][lane + LP * q] = acc[i][q];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < SOM_BLEND_J * d; e += blockDim.x) {
        const int i = e / d, t = e % d, j = j0 + i;
        if (j >= g || (frozen && frozen[j])) continue;
        double num = 0.0, dn = 0.0;
#pragma unroll 8
        for (int w = 0; w < NG; ++w) {
            num += red[w][i][t];
            dn += rden[w][i];
        }
        const double Lj = (double)L[(size_t)j * d + t];
        L[(size_t)j * d + t] = (float)(Lj + (double)alpha / (double)B * (num - dn * Lj));
    }
}

// Whether a step of this shape takes the direct path: the FP64 distances run at
// about 10^13 a second, so 2^29 of them (53 us) stay below the general path's
// launches; the blend reads the whole batch for every two landmarks, which
// 4096 points keep under its other costs, and holds their weights for all g
// landmarks beside the batch in LDS (64 + 32 KB at the limits).
bool som_direct(int B, int g, int d) {
    return B <= SOM_DIRECT_BATCH && g <= SOM_DIRECT_G && (int64_t)B * g * d <= ((int64_t)1 << 29);
}

hipError_t launch_som_direct(const float *X, int64_t n, int64_t ldx, int d, float *L, const float *l2d, int g,
                             const int32_t *rows, int B, int32_t *nearest, float sigma, float alpha,
                             const uint8_t *frozen, hipStream_t s) {
    // more points per wavefront only once that many blocks fill the chip
    const int pw = B <= 1024 ? 1 : B <= 2048 ? 2 : 4;
    const int per = SOM_WAVES * pw;
    const int tr = d <= 64 ? 4 : 1;
    const size_t smem = sizeof(double) * per * d + sizeof(float) * 64 * tr * (d | 1);
    auto bmu = tr == 4 ? (pw == 1 ? som_bmu<1, 4> : pw == 2 ? som_bmu<2, 4> : som_bmu<4, 4>)
                       : (pw == 1 ? som_bmu<1, 1> : pw == 2 ? som_bmu<2, 1> : som_bmu<4, 1>);
    hipLaunchKernelGGL(bmu, dim3((B + per - 1) / per), dim3(64 * SOM_WAVES), smem, s, X, n, ldx, d, L, g, rows, B,
                       nearest);
    auto blend = d <= 16 ? som_blend<16, 1, 16> : d <= 32 ? som_blend<32, 1, 16> : d <= 64 ? som_blend<64, 1, 16>
                : d <= 128 ? som_blend<64, 2, 8> : som_blend<64, 4, 4>;
    hipLaunchKernelGGL(blend, dim3((g + SOM_BLEND_J - 1) / SOM_BLEND_J), dim3(d <= 64 ? 1024 : d <= 128 ? 512 : 256),
                       sizeof(double) * SOM_BLEND_J * g + sizeof(int2) * B, s, X, ldx, d, L, l2d, g, rows, nearest, B,
                       sigma, alpha, frozen);
    return hipGetLastError();
}

// Lexicographic order on (squared distance, index).
__device__ __forceinline__ bool lex_before(double a, int ia, double b, int ib) {
    return a < b || (a == b && ia < ib);
}

// One wavefront per added landmark q at 2-D position p_q:
//  1. its kfit nearest 2-D landmarks by (squared distance, index), one per
//     round: each round takes the wave-wide lexicographic minimum among the
//     landmarks that come after the previous round's choice;
//  2. weights w_i = exp(-(d2_i - d2_1) / (2 sigma^2)) (scaled so the nearest
//     weighs 1) and the 3 x 3 weighted normal matrix G of the affine fit
//     z -> A z + c, z = (lx, ly, 1), in FP64 wave sums;
//  3. v = G^-1 (p, 1) by Cramer's rule and coefficients beta_i = w_i (v . z_i),
//     or the weighted mean when G is numerically singular (fewer than three
//     or collinear neighbours);
//  4. out_q = sum_i beta_i L_i, lanes over dimensions.
constexpr int FIT_MAX_K = 64;

__global__ void __launch_bounds__(64) fit_landmarks(const float *__restrict__ L, const float *__restrict__ l2d,
                                                    int g, int d, const float *__restrict__ p, int kfit,
                                                    float sigma, float *__restrict__ out) {
    __shared__ double beta[FIT_MAX_K];
    __shared__ int nbs[FIT_MAX_K];
    const int q = blockIdx.x;
    const int lane = threadIdx.x;
    const double px = (double)p[2 * q], py = (double)p[2 * q + 1];
    double prev_d = -1.0;
    int prev_j = -1;
    double my_d = 0.0;  // lane i keeps neighbour i
    int my_j = -1;
    for (int r = 0; r < kfit; ++r) {
        double bd = INFINITY;
        int bj = 0x7fffffff;
        for (int j = lane; j < g; j += 64) {
            const double dx = (double)l2d[2 * j] - px, dy = (double)l2d[2 * j + 1] - py;
            const double dj = dx * dx + dy * dy;
            if (lex_before(prev_d, prev_j, dj, j) && lex_before(dj, j, bd, bj)) {
                bd = dj;
                bj = j;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double od = __shfl_xor(bd, o);
            const int oj = __shfl_xor(bj, o);
            if (lex_before(od, oj, bd, bj)) {
                bd = od;
                bj = oj;
            }
        }
        prev_d = bd;
        prev_j = bj;
        if (lane == r) {
            my_d = bd;
            my_j = bj;
        }
    }
    const double d0 = __shfl(my_d, 0);
    const bool act = lane < kfit;
    const double w = act ? exp(-(my_d - d0) / (2.0 * (double)sigma * (double)sigma)) : 0.0;
    const double zx = act ? (double)l2d[2 * my_j] : 0.0, zy = act ? (double)l2d[2 * my_j + 1] : 0.0;
    double Gs[7] = {w * zx * zx, w * zx * zy, w * zx, w * zy * zy, w * zy, w, 0.0};
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) Gs[i] += __shfl_xor(Gs[i], o);
    const double G[3][3] = {{Gs[0], Gs[1], Gs[2]}, {Gs[1], Gs[3], Gs[4]}, {Gs[2], Gs[4], Gs[5]}};
    const double W = Gs[5];
    auto det3 = [](const double (&M)[3][3]) {
        return M[0][0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) - M[0][1] * (M[1][0] * M[2][2] - M[1][2] * M[2][0]) +
               M[0][2] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]);
    };
    const double det = det3(G);
    const double md = (G[0][0] + G[1][1] + G[2][2]) / 3.0;
    double bt;
    if (kfit >= 3 && det > 1e-12 * md * md * md) {
        const double e[3] = {px, py, 1.0};
        double v[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double M[3][3];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) M[a][b] = (b == c) ? e[a] : G[a][b];
            v[c] = det3(M) / det;
        }
        bt = w * (v[0] * zx + v[1] * zy + v[2]);
    } else {
        bt = w / W;
    }
    if (act) {
        beta[lane] = bt;
        nbs[lane] = my_j;
    }
    __syncthreads();
    for (int c = lane; c < d; c += 64) {
        double o = 0.0;
        for (int i = 0; i < kfit; ++i) o += beta[i] * (double)L[(size_t)nbs[i] * d + c];
        out[(size_t)q * d + c] = (float)o;
    }
}

hipError_t launch_fit_landmarks(const float *L, const float *l2d, int g, int d, const float *p, int m,
                                int kfit, float sigma, float *out, hipStream_t s) {
    if (m > 0)
        hipLaunchKernelGGL(fit_landmarks, dim3((unsigned)m), dim3(64), 0, s, L, l2d, g, d, p, kfit, sigma, out);
    return hipGetLastError();
}

}  // namespace esom
