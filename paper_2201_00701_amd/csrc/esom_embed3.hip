// EmbedSOM projection into 3-D (the paper states the method in 2-D for
// brevity, Section "Landmark-directed dimensionality reduction"): the same
// neighbours, scores and segment projections, with 3-D landmark positions l
// (g x 3) and a 3 x 3 system solved by Cramer's rule.  The k nearest
// landmarks come from the 2-D path's screen and exact selection (k-NN only);
// this kernel then works in FP64 throughout (list_project.h).
// Bound by FP64 arithmetic and the latency of a point's serial chain.  A
// wavefront per point with its sums over 64 lanes by shuffles and every pair
// projected from the rows took 2605 us for 200k points (32-D, 400 landmarks, k =
// 16); 16 lanes a point with the pair table take 177 us.
#include "list_project.h"

namespace esom {

template <int G>
__global__ void __launch_bounds__(LP_THREADS) embed3_kernel(ListArgs e) {
    extern __shared__ __align__(16) unsigned char lsm[];
    LpNeighbour *nb = reinterpret_cast<LpNeighbour *>(lsm) + (threadIdx.x & ~(G - 1));
    unsigned short *pairs = reinterpret_cast<unsigned short *>(reinterpret_cast<LpNeighbour *>(lsm) + LP_THREADS);
    lp_pairs(pairs, e.use_cutoff ? e.k - 1 : e.k);
    constexpr int PW = 64 / G;  // points per wavefront
    const int64_t wave = (int64_t)blockIdx.x * (LP_THREADS / 64) + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * (LP_THREADS / 64);
    for (int64_t p0 = wave * PW; p0 < e.n; p0 += nw * PW) {
        const int64_t pi = p0 + (threadIdx.x & 63) / G;
        lp_point<G, 3>(e, pi, pi < e.n, nb, pairs);
    }
}

// tab[u][v] = 1 / (2 |L_u - L_v|^2) in FP64 by landmark positions, 0 for
// coincident landmarks: 16 x 16 pairs a block from two slices of the padded rows
// in LDS.
constexpr int TAB_TILE = 16;

__global__ void __launch_bounds__(256) pair_table64(const float *__restrict__ Lpad, int g, int dp,
                                                    double *__restrict__ tab) {
    extern __shared__ __align__(16) float tsm[];
    const int rs = dp + 1;
    float *Lu = tsm, *Lv = tsm + TAB_TILE * rs;
    const int u0 = blockIdx.y * TAB_TILE, v0 = blockIdx.x * TAB_TILE;
    for (int e = threadIdx.x; e < TAB_TILE * dp; e += blockDim.x) {
        const int r = e / dp, q = e % dp;
        Lu[r * rs + q] = u0 + r < g ? Lpad[(size_t)(u0 + r) * dp + q] : 0.f;
        Lv[r * rs + q] = v0 + r < g ? Lpad[(size_t)(v0 + r) * dp + q] : 0.f;
    }
    __syncthreads();
    const int ty = threadIdx.x / TAB_TILE, tx = threadIdx.x % TAB_TILE;
    if (u0 + ty >= g || v0 + tx >= g) return;
    double s = 0.0;
#pragma unroll 8
    for (int q = 0; q < dp; ++q) {
        const double df = (double)Lv[tx * rs + q] - (double)Lu[ty * rs + q];
        s = fma(df, df, s);
    }
    tab[(size_t)(u0 + ty) * g + v0 + tx] = s > 0.0 ? 0.5 / s : 0.0;
}

// The table pays once the points read its g^2 entries several times over; its
// size is kept to 32 MB.
size_t embed3_table_bytes(int64_t n, int g, int k) {
    const int64_t reads = n * k * (k - 1) / 2;
    return g <= 2048 && reads > 4 * (int64_t)g * g ? sizeof(double) * (size_t)g * g : 0;
}

hipError_t launch_embed3(const ListArgs &e, double *tab, int num_cus, hipStream_t s) {
    ListArgs a = e;
    a.tab = tab;
    if (tab) {
        const unsigned t = (unsigned)((e.g + TAB_TILE - 1) / TAB_TILE);
        hipLaunchKernelGGL(pair_table64, dim3(t, t), dim3(256), sizeof(float) * 2 * TAB_TILE * (e.dp + 1), s, e.Lpad,
                           e.g, e.dp, tab);
    }
    const int gl = e.k <= 16 ? 16 : e.k <= 32 ? 32 : 64;
    const long long per = (long long)(LP_THREADS / gl);
    long long blocks = (e.n + per - 1) / per;
    if (blocks > (long long)num_cus * 8) blocks = (long long)num_cus * 8;
    if (blocks < 1) blocks = 1;
    auto kern = gl == 16 ? embed3_kernel<16> : gl == 32 ? embed3_kernel<32> : embed3_kernel<64>;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(LP_THREADS), lp_lds_bytes(e.k), s, a);
    return hipGetLastError();
}

}  // namespace esom
