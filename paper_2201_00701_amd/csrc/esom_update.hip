// Batch landmark update: nearest-landmark sums and counts, then a k-means or
// batch-SOM blend (semi-supervised model update of the paper's supervision
// section, in data-parallel batch form).
//
// The rows stream once into FP64 sums kept in LDS (upd_accum), and the blocks'
// sums are added (upd_reduce).  FP64 sums make the result independent of the
// visiting order up to FP64 rounding, far below the FP32 output rounding.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "esom_internal.h"

namespace esom {

constexpr int UPD_BLOCK = 256;

// Sums of the rows by nearest landmark in LDS.  The landmarks go in groups whose
// gg x d FP64 sums fit in LDS, the points in P ranges; a block takes one group and
// one range.  Each wavefront takes 64 points at a time, lists those of its group
// (their order in memory, so the blocks of a range read its rows as one stream),
// and adds the rows with LDS atomics, LP lanes a row (LP >= d up to 64, NQ
// dimensions a lane beyond), ACC_U loads in flight.  Blocks 8 apart (the same XCD)
// take the groups of one range.  The partial array of a range is [g][d + 1], the
// count last.
// Bound by the LDS atomics, which take an FP64 lane a clock (10M x 64-D: 2.5M
// adds per CU, 1.0 ms; the row stream alone takes 0.55).  10M x 64-D, 1024
// landmarks: a counting sort of all points and one block per 4096 points of a
// landmark took 2.41 ms (sums 1.94, scatter 0.33, histogram 0.13); ranges sorted
// in LDS and summed in registers 1.70 ms (rows gathered in random order, 1.9
// TB/s); this 1.75 ms with upd_compact, and for every landmark count.  1M x 32-D,
// 400 landmarks: 0.36 ms by the sort, now 0.063 ms.
constexpr int ACC_BLOCK = 1024;
constexpr int ACC_U = 16;                           // row loads in flight per LP lanes (divided by NQ)
constexpr int ACC_RANGE = 1024;                     // points per range at least
constexpr int ACC_BLOCKS = 256;                     // blocks at most (one per CU)
constexpr size_t ACC_LDS_BYTES = (size_t)148 << 10;  // sums and counts of a group

__device__ __forceinline__ void lds_add_f64(double *p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <int LP, int NQ>
__global__ void __launch_bounds__(ACC_BLOCK) upd_accum(const float *__restrict__ X, int64_t n, int64_t ldx, int d,
                                                       const int32_t *__restrict__ nearest, int64_t ld, int g,
                                                       int gg, int groups, int P, double *__restrict__ partial) {
    extern __shared__ __align__(16) unsigned char asm_[];
    __shared__ int2 lists[ACC_BLOCK / 64][64];
    const int grp = (blockIdx.x / 8) % groups, rng = (blockIdx.x / (8 * groups)) * 8 + blockIdx.x % 8;
    if (rng >= P) return;
    const int j0 = grp * gg, gn = g - j0 < gg ? g - j0 : gg;  // this group's landmarks
    double *acc = reinterpret_cast<double *>(asm_);           // gn x d
    int *cnt = reinterpret_cast<int *>(acc + (size_t)gg * d);
    const int tid = threadIdx.x, lane64 = tid & 63, wv = tid >> 6, lane = lane64 % LP, sub = lane64 / LP;
    for (int e = tid; e < gn * d; e += ACC_BLOCK) acc[e] = 0.0;
    for (int e = tid; e < gn; e += ACC_BLOCK) cnt[e] = 0;
    __syncthreads();
    constexpr int PP = 64 / LP, U = ACC_U / NQ;
    int2 *list = lists[wv];
    const int64_t per = ((n + P - 1) / P + 63) & ~(int64_t)63;
    const int64_t r0 = rng * per, r1 = r0 + per < n ? r0 + per : n;
    int64_t i = r0 + 64 * wv + lane64;
    int jn = i < r1 ? nearest[i * ld] : -1;
    for (int64_t ib = r0 + 64 * wv; ib < r1; ib += ACC_BLOCK) {
        const int j = jn - j0;
        const bool in = jn >= 0 && jn < g && j >= 0 && j < gn;  // indices outside [0, g) are ignored
        const unsigned long long mk = __ballot(in);
        const int m = __popcll(mk);
        if (in) {
            list[__popcll(mk & ((1ull << lane64) - 1ull))] = make_int2((int)(i - r0), j);
            atomicAdd(&cnt[j], 1);
        }
        i += ACC_BLOCK;
        jn = i < r1 ? nearest[i * ld] : -1;  // the next 64 points' landmarks
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int p0 = 0; p0 < m; p0 += U * PP) {
            int jj[U];
            float x[U][NQ];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int at = p0 + u * PP + sub;
                const int2 pt = list[at < m ? at : 0];
                jj[u] = at < m ? pt.y : -1;
                const float *xr = X + (r0 + pt.x) * ldx;
#pragma unroll
                for (int q = 0; q < NQ; ++q) x[u][q] = at < m && lane + LP * q < d ? xr[lane + LP * q] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    if (jj[u] >= 0 && lane + LP * q < d) lds_add_f64(&acc[jj[u] * d + lane + LP * q], (double)x[u][q]);
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    double *out = partial + ((size_t)rng * g + j0) * (d + 1);
    for (int j = tid / LP; j < gn; j += ACC_BLOCK / LP) {
        for (int t = lane; t < d; t += LP) out[(size_t)j * (d + 1) + t] = acc[j * d + t];
        if (lane == 0) out[(size_t)j * (d + 1) + d] = (double)cnt[j];
    }
}

// near[i] = nearest[i * ld]: every group would read a strided list's lines again.
__global__ void upd_compact(const int32_t *__restrict__ nearest, int64_t ld, int64_t n, int32_t *__restrict__ near) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) near[i] = nearest[i * ld];
}

// Adds the P partial sums of landmark j = blockIdx.x, the threads sharing the
// partials of each of the d + 1 columns; then the k-means blend (kind 0) or the
// sums for the topology blend (S).
__global__ void __launch_bounds__(UPD_BLOCK) upd_reduce(const double *partial, int P, int g, int d, int kind,
                                                        float alpha, float *__restrict__ L, double *S,
                                                        int32_t *__restrict__ counts_out) {
    __shared__ double red[UPD_BLOCK + ESOM_MAX_D + 1];  // share x column
    const int j = blockIdx.x;
    const int cols = d + 1;
    const int ns = cols < UPD_BLOCK ? UPD_BLOCK / cols : 1;  // shares
    for (int e = threadIdx.x; e < ns * cols; e += UPD_BLOCK) {
        const int sh = e / cols, t = e % cols;
        double s = 0.0;
#pragma unroll 16
        for (int p = sh; p < P; p += ns) s += partial[((size_t)p * g + j) * cols + t];
        red[e] = s;
    }
    __syncthreads();
    auto total = [&](int t) {
        double s = 0.0;
        for (int sh = 0; sh < ns; ++sh) s += red[sh * cols + t];
        return s;
    };
    const double den = total(d);
    if (counts_out && threadIdx.x == 0) counts_out[j] = (int32_t)den;
    for (int t = threadIdx.x; t < cols; t += blockDim.x) {
        if (kind != 0) {
            S[(size_t)j * cols + t] = total(t);
        } else if (t < d && den > 0.0) {
            const double Lj = (double)L[(size_t)j * d + t];
            L[(size_t)j * d + t] = (float)(Lj + (double)alpha * (total(t) / den - Lj));
        }
    }
}

// Blends over the 2-D topology, L_j from sum_b h_jb (S_b, c_b).  kind 1: batch
// SOM; kind 2: one online SOM step over a batch of `batch` points, the average
// of the single-point online updates
//   L_j += (alpha / batch) sum_b h_jb (S_b - c_b L_j),
// skipping landmarks with frozen[j] != 0.  A block takes BLEND_J landmarks j and
// walks the landmarks b in chunks of BLEND_B: its threads form the chunk's
// BLEND_J x BLEND_B weights in LDS (one exponential each), then each wavefront
// adds its share of the chunk's rows, lanes over the d + 1 columns of S (the
// count is the last), and the wavefronts' sums meet in LDS.
// Bound by the latency of the chunk steps; two landmarks a block keep 200
// blocks in flight at g = 400.  400 landmarks, 32-D: every thread used to
// evaluate all g exponentials for itself, twice, 287 us; now 13 us.
constexpr int BLEND_J = 2;
constexpr int BLEND_B = UPD_BLOCK / BLEND_J;

template <int NQ>
__global__ void __launch_bounds__(UPD_BLOCK) upd_blend(const double *__restrict__ sums, const float *__restrict__ l2d,
                                                       int g, int d, int kind, float alpha, float sigma,
                                                       float *__restrict__ L, const uint8_t *__restrict__ frozen,
                                                       int64_t batch) {
    constexpr int NW = UPD_BLOCK / 64;
    __shared__ double h[BLEND_J][BLEND_B];
    __shared__ double red[NW][BLEND_J][64 * NQ];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int j0 = blockIdx.x * BLEND_J;
    const int cols = d + 1;
    const double s2 = 2.0 * (double)sigma * (double)sigma;
    const int hj = threadIdx.x / BLEND_B, hb = threadIdx.x % BLEND_B;
    const int jh = min(j0 + hj, g - 1);
    const double jx = (double)l2d[2 * jh], jy = (double)l2d[2 * jh + 1];
    double acc[BLEND_J][NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int i = 0; i < BLEND_J; ++i) acc[i][q] = 0.0;
    for (int b0 = 0; b0 < g; b0 += BLEND_B) {
        __syncthreads();
        const int bh = b0 + hb;
        double w = 0.0;
        if (bh < g) {
            if (sigma == 0.f) {
                w = bh == jh ? 1.0 : 0.0;
            } else {
                const double dx = jx - (double)l2d[2 * bh], dy = jy - (double)l2d[2 * bh + 1];
                w = exp(-(dx * dx + dy * dy) / s2);
            }
        }
        h[hj][hb] = w;
        __syncthreads();
        const int nb = g - b0 < BLEND_B ? g - b0 : BLEND_B;
#pragma unroll 8
        for (int b = wv; b < nb; b += NW) {
            const double *Sb = sums + (size_t)(b0 + b) * cols;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int t = lane + 64 * q;
                const double v = t < cols ? Sb[t] : 0.0;
#pragma unroll
                for (int i = 0; i < BLEND_J; ++i) acc[i][q] = fma(h[i][b], v, acc[i][q]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int i = 0; i < BLEND_J; ++i) red[wv][i][lane + 64 * q] = acc[i][q];
    __syncthreads();
    for (int e = threadIdx.x; e < BLEND_J * d; e += UPD_BLOCK) {
        const int i = e / d, t = e % d, j = j0 + i;
        if (j >= g || (kind == 2 && frozen && frozen[j])) continue;
        double num = 0.0, den = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            num += red[w][i][t];
            den += red[w][i][d];
        }
        const double Lj = (double)L[(size_t)j * d + t];
        if (kind == 2)
            L[(size_t)j * d + t] = (float)(Lj + (double)alpha / (double)batch * (num - den * Lj));
        else if (den > 0.0)
            L[(size_t)j * d + t] = (float)(Lj + (double)alpha * (num / den - Lj));
    }
}

static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

// Landmark groups of a shape.
static int acc_group(int g, int d) {
    const int gg = (int)(ACC_LDS_BYTES / (sizeof(double) * d + sizeof(int)));
    const int groups = (g + gg - 1) / gg;
    return (g + groups - 1) / groups;
}
static int acc_groups(int g, int d) { return (g + acc_group(g, d) - 1) / acc_group(g, d); }

// The ranges n points go in: with the groups enough blocks to fill the chip once,
// each range of at least ACC_RANGE points, as many as there is room for (with the
// sums of 3 ranges 100k points x 32-D, 400 landmarks, take 411 us, of all 98 ranges
// 32).  One range needs no partial array beside the sums.  The compact copy comes
// after the ranges.
UpdatePlan update_plan(int64_t n, int g, int d, int64_t nearest_ld, size_t room) {
    const size_t sums = sizeof(double) * (size_t)g * (d + 1);
    UpdatePlan u;
    int64_t r = (n + ACC_RANGE - 1) / ACC_RANGE;
    if (r > ACC_BLOCKS / acc_groups(g, d)) r = ACC_BLOCKS / acc_groups(g, d);
    const int64_t most = room > al256(sums) + 255 ? (int64_t)((room - al256(sums) - 255) / sums) : 0;
    if (r > most) r = most;
    u.ranges = r < 1 ? 1 : (int)r;
    u.bytes = al256(sums) + (u.ranges > 1 ? al256(sums * u.ranges) : 0);
    const size_t copy = al256(sizeof(int32_t) * (size_t)(n > 0 ? n : 1));
    u.compact = n > 0 && acc_groups(g, d) > 1 && nearest_ld > 1 && room > u.bytes && room - u.bytes >= copy;
    if (u.compact) u.bytes += copy;
    return u;
}

hipError_t launch_update(const UpdateArgs &u, void *ws, const UpdatePlan &plan, hipStream_t s) {
    const size_t sb = sizeof(double) * (size_t)u.g * (u.d + 1);
    char *p = static_cast<char *>(ws);
    double *sums = reinterpret_cast<double *>(p), *partial = sums;
    p += al256(sb);
    const int ranges = plan.ranges;
    if (ranges > 1) {
        partial = reinterpret_cast<double *>(p);
        p += al256(sb * ranges);
    }
    const int32_t *near = u.nearest;
    int64_t ld = u.nearest_ld;
    if (plan.compact) {
        int32_t *c = reinterpret_cast<int32_t *>(p);
        hipLaunchKernelGGL(upd_compact, dim3((unsigned)((u.n + 255) / 256)), dim3(256), 0, s, near, ld, u.n, c);
        near = c;
        ld = 1;
    }
    const int gg = acc_group(u.g, u.d), groups = acc_groups(u.g, u.d);
    const size_t sh = (sizeof(double) * u.d + sizeof(int)) * (size_t)gg;
    auto acc = u.d <= 16 ? upd_accum<16, 1> : u.d <= 32 ? upd_accum<32, 1> : u.d <= 64 ? upd_accum<64, 1>
              : u.d <= 128 ? upd_accum<64, 2> : upd_accum<64, 4>;
    hipLaunchKernelGGL(acc, dim3((ranges + 7) / 8 * 8 * groups), dim3(ACC_BLOCK), sh, s, u.X, u.n, u.ldx, u.d, near,
                       ld, u.g, gg, groups, ranges, partial);
    // (one range: reduced in place for the topology blends)
    hipLaunchKernelGGL(upd_reduce, dim3(u.g), dim3(UPD_BLOCK), 0, s, partial, ranges, u.g, u.d, u.kind, u.alpha, u.L,
                       sums, u.counts);
    if (u.kind != 0) {
        auto kern = u.d < 64 ? upd_blend<1> : u.d < 128 ? upd_blend<2> : upd_blend<5>;
        hipLaunchKernelGGL(kern, dim3((u.g + BLEND_J - 1) / BLEND_J), dim3(UPD_BLOCK), 0, s, sums, u.l2d, u.g, u.d,
                           u.kind, u.alpha, u.sigma, u.L, u.frozen, u.batch);
    }
    return hipGetLastError();
}

}  // namespace esom
