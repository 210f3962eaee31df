// The materialised-distance path: the distance pass and the k-NN selection
// as two kernels with the keys written to device memory between them (the
// separation the paper's "k-NN step" weighs against fusion and leaves for
// extreme d).  It serves the dimensions beyond the fused kernel's register
// budget (d above 64 in FP32 mode, above 128 in BF16 mode, up to 256), which
// otherwise go point by point through the exact FP64 path.
//
//   keys_kernel    one block per 64 points: their centred rows staged in LDS,
//                  the wavefronts share out the 32-landmark tiles of the FP32 MFMA
//                  operand (v_mfma_f32_32x32x2f32, C initialised to |L_j - c|^2),
//                  key_ij = |L_j - c|^2 - 2 <x_i - c, L_j - c> for all landmarks,
//                  stored per point in the order the accumulators hold them;
//   select_kernel  one wavefront per point: the threshold tau is the C-th
//                  smallest of the 64 lanes' key minima, so at least C keys lie
//                  within it; these candidates are rescored with exact FP32
//                  differences and ranked by (distance, index); the point is
//                  certified when its k-th rescored distance lies below tau by
//                  more than the keys' rounding bound, else it is marked for the
//                  exact path, as are a k-th / (k+1)-th tie FP32 cannot order and a
//                  point with more than 64 candidates.
// The projection then runs from these neighbours (embed_project) and the
// exact path takes the marked points.
#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "embed_kernel.h"
#include "esom_internal.h"

namespace esom {

constexpr int MK_WAVES = 4;   // wavefronts per keys block
constexpr int MK_POINTS = 64;  // points per keys block

// Order in which a point's keys are stored: tile t, lane half h, accumulator
// register r at 32 t + 16 h + r, which is landmark position 64 (t / 2) + 32 (t
// mod 2) + 2 r + h.
__device__ __forceinline__ int key_position(int e) {
    return 64 * (e >> 6) + 32 * ((e >> 5) & 1) + 2 * (e & 15) + ((e >> 4) & 1);
}

// Bound by the FP32 MFMA rate: an A load serves both 32-point halves, and the
// accumulators leave in 64-byte pieces.  50k points x 100-D, 400 landmarks: 254 us
// with one 32-point half a wavefront and its keys stored one by one, now 83 us.
__global__ void __launch_bounds__(64 * MK_WAVES) keys_kernel(MatArgs m) {
    extern __shared__ __align__(16) float xs[];  // 64 centred rows, stride dp + 1
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int h = lane >> 5, i32 = lane & 31;
    const int dp = m.dp, rs = dp + 1;
    const int64_t p0 = (int64_t)blockIdx.x * MK_POINTS;
    for (int r = wv; r < MK_POINTS; r += MK_WAVES) {
        const int64_t pi = p0 + r < m.n ? p0 + r : m.n - 1;
        for (int c = lane; c < dp; c += 64) xs[r * rs + c] = c < m.d ? m.X[pi * m.ldx + c] - m.cent[c] : 0.f;
    }
    __syncthreads();
    const float *x0 = xs + i32 * rs + 8 * h, *x1 = x0 + 32 * rs;  // MFMA step s: dimension 16 (s / 8) + 8 h + s % 8
    for (int t = wv; t < m.ntiles; t += MK_WAVES) {
        f32x16 acc[2];
        const float4 *np = reinterpret_cast<const float4 *>(m.norms + (size_t)(t * 2 + h) * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = np[q];
            acc[0][4 * q] = v.x;
            acc[0][4 * q + 1] = v.y;
            acc[0][4 * q + 2] = v.z;
            acc[0][4 * q + 3] = v.w;
        }
        acc[1] = acc[0];
        const float *At = static_cast<const float *>(m.A) + (size_t)t * (dp / 2) * 64 + lane;
        for (int s0 = 0; s0 < dp / 2; s0 += 8) {  // dp is a multiple of 16
            float av[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) av[s] = At[(size_t)(s0 + s) * 64];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s], x0[2 * s0 + s], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s], x1[2 * s0 + s], acc[1], 0, 0, 0);
            }
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int64_t pi = p0 + 32 * p + i32;
            if (pi < m.n) {
                float4 *k4 = reinterpret_cast<float4 *>(m.keys + pi * m.gpad + 32 * t + 16 * h);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    k4[q] = make_float4(acc[p][4 * q], acc[p][4 * q + 1], acc[p][4 * q + 2], acc[p][4 * q + 3]);
            }
        }
    }
}

// An unsigned whose order is the float's.
__device__ __forceinline__ unsigned float_order(float f) {
    const unsigned u = __float_as_uint(f);
    return u ^ ((unsigned)((int)u >> 31) | 0x80000000u);
}

// NK: keys per lane at most (gpad <= 64 NK).  Bound by the instructions of the
// rescoring and ranking.  50k points x 100-D, 400 landmarks, k = 16: 1068 us with
// 40-entry insertion lists per lane and C + 1 rounds of shuffled minima, now
// 165 us.
template <int NK>
__global__ void __launch_bounds__(256) select_kernel(MatArgs m) {
    __shared__ int cpos[4][64];  // per wavefront: candidate positions
    __shared__ float cd[4][64];  // ... the rescored candidates, ranked
    __shared__ int cj[4][64];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t nw = (int64_t)gridDim.x * 4;
    const int C = m.C, k = m.k;
    for (int64_t pi = (int64_t)blockIdx.x * 4 + wv; pi < m.n; pi += nw) {
        const float *krow = m.keys + pi * m.gpad;
        float key[NK];
        float mv = INFINITY;
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            key[i] = 64 * i < m.gpad ? krow[64 * i + lane] : INFINITY;
            mv = fminf(mv, key[i]);
        }
        // the C-th smallest of the lanes' minima, by bisection on its bits
        const unsigned om = float_order(mv);
        unsigned lo = 0u;  // fewer than C minima lie below lo
#pragma unroll
        for (int b = 31; b >= 0; --b) {
            const unsigned mid = lo | (1u << b);
            if (__popcll(__ballot(om < mid)) < C) lo = mid;
        }
        const unsigned long long le = __ballot(om == lo);  // the lanes that hold it
        const float tau = __shfl(mv, le ? __builtin_ctzll(le) : 0);
        // candidates
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            const bool in = key[i] <= tau && key[i] < INFINITY;  // padded keys are +inf
            const unsigned long long mk = __ballot(in);
            const int at = cnt + __popcll(mk & ((1ull << lane) - 1ull));
            if (in && at < 64) cpos[wv][at] = key_position(64 * i + lane);
            cnt += __popcll(mk);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const bool over = cnt > 64;
        const int nc = over ? 64 : cnt;
        const bool act = lane < nc;
        const int pos = act ? cpos[wv][lane] : 0;
        const int jl = act ? m.perm[pos] : INT32_MAX;
        // exact FP32 rescoring, the four lanes of a quad on one candidate at a
        // time (64 consecutive bytes of 16 rows per load); |x - c|^2 along the way
        const float *x = m.X + pi * m.ldx;
        float sum[4] = {0.f, 0.f, 0.f, 0.f}, xn = 0.f;
        {
            const char *base = reinterpret_cast<const char *>(m.Lpad);
            const unsigned off = (unsigned)pos * (unsigned)m.dp * 4u, lo16 = 16u * (lane & 3);
            const unsigned o[4] = {(unsigned)quad_bcast<0>((int)off) + lo16, (unsigned)quad_bcast<1>((int)off) + lo16,
                                   (unsigned)quad_bcast<2>((int)off) + lo16, (unsigned)quad_bcast<3>((int)off) + lo16};
            for (int c = 0; c < m.dp / 16; ++c) {
                float4 lv[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    lv[q] = *reinterpret_cast<const float4 *>(base + (size_t)(o[q] + 64u * c));
                const int t0 = 16 * c + 4 * (lane & 3);
                float xv[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) xv[t] = t0 + t < m.d ? x[t0 + t] : 0.f;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float v = t0 + t < m.d ? xv[t] - m.cent[t0 + t] : 0.f;
                    xn = fmaf(v, v, xn);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float e0 = xv[0] - lv[q].x, e1 = xv[1] - lv[q].y, e2 = xv[2] - lv[q].z, e3 = xv[3] - lv[q].w;
                    sum[q] = fmaf(e0, e0, sum[q]);
                    sum[q] = fmaf(e1, e1, sum[q]);
                    sum[q] = fmaf(e2, e2, sum[q]);
                    sum[q] = fmaf(e3, e3, sum[q]);
                }
            }
        }
        xn = quad_sum(xn);  // every quad has all dimensions
        float d2 = INFINITY;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float t = quad_sum(sum[q]);
            d2 = (lane & 3) == q ? t : d2;
        }
        if (!act) d2 = INFINITY;
        // rank by (distance, landmark index)
        int rank = 0;
        for (int p = 0; p < nc; ++p) {
            const float dp2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(d2), p));
            const int jp = __builtin_amdgcn_readlane(jl, p);
            rank += (dp2 < d2 || (dp2 == d2 && jp < jl)) ? 1 : 0;
        }
        cd[wv][lane] = INFINITY;
        cj[wv][lane] = INT32_MAX;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (act) {
            cd[wv][rank] = d2;
            cj[wv][rank] = jl;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // certificate: every non-candidate's key is > tau, so its exact
        // distance^2 exceeds tau + |x - c|^2 - E (E the FP32 keys' rounding bound)
        const float lmax = m.lmax[0];
        const float sx = sqrtf(xn);
        const float facc = (2.f * m.dp + 16.f) * U32 * (sx + lmax) * (sx + lmax);
        const float E = 1.01f * (2.f * (2.f * U32 + U32 * U32) * sx * lmax + facc);
        float rhs = tau + xn - E;
        rhs -= 4.f * U32 * (fabsf(tau) + xn + E);
        const float d2r = cd[wv][lane];
        const float d2k = cd[wv][k - 1];
        const float d2k1 = k < 64 ? cd[wv][k] : INFINITY;
        const float rb = (float)(m.dp + 3) * U32;  // rounding bound of a rescored distance
        // (all g landmarks candidates: nothing is left out)
        bool mark = over || !(cnt < m.g ? d2k * (1.f + rb) < rhs : d2k < INFINITY);
        if (d2k1 < INFINITY && d2k1 - d2k <= 2.f * rb * d2k1) mark = true;  // k-th / (k+1)-th closer than FP32 orders
        // adjacent entries FP32 cannot order when the caller wants the exact order
        bool order = false;
        if (m.exact_order) {
            const float prev = __shfl_up(d2r, 1);
            order = __ballot(lane > 0 && lane < k && d2r - prev <= 2.f * rb * d2r) != 0ull;
        }
        if (lane < k) {
            m.knn_idx[pi * k + lane] = cj[wv][lane];
            m.knn_d2[pi * k + lane] = d2r;
        }
        if (lane == 0) m.knn_mark[pi] = mark ? 1 : order ? 2 : 0;
        __builtin_amdgcn_wave_barrier();
    }
}

hipError_t launch_materialise(const MatArgs &m, int num_cus, hipStream_t s) {
    const unsigned kblocks = (unsigned)((m.n + MK_POINTS - 1) / MK_POINTS);
    const size_t ksmem = sizeof(float) * (size_t)MK_POINTS * (m.dp + 1);
    hipLaunchKernelGGL(keys_kernel, dim3(kblocks), dim3(64 * MK_WAVES), ksmem, s, m);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    long long sblocks = (m.n + 3) / 4;
    if (sblocks > (long long)num_cus * 8) sblocks = (long long)num_cus * 8;
    if (sblocks < 1) sblocks = 1;
    auto sel = m.gpad <= 256 ? select_kernel<4> : m.gpad <= 512 ? select_kernel<8> : m.gpad <= 1024 ? select_kernel<16>
              : m.gpad <= 2048 ? select_kernel<32> : select_kernel<64>;
    hipLaunchKernelGGL(sel, dim3((unsigned)sblocks), dim3(256), 0, s, m);
    return hipGetLastError();
}

}  // namespace esom
