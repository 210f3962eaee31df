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

#include <string.h>

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

// Points of a 2-D call whose neighbours are certain but closer than FP32 orders
// (listed from the end of the fallback arrays): their lists ranked by exact
// distance and the points projected again.  The exact path used to take them with
// all others and formed the distances to all landmarks: in the 10M x 64-D frame
// (1024 landmarks, k = 16) 2.30 ms for its 1.1% of the points; now 0.57 ms here and
// 0.30 ms there for the others.
template <int G>
__global__ void __launch_bounds__(LP_THREADS) embed_reorder(ListArgs e, const int32_t *__restrict__ list, int64_t cap,
                                                            unsigned long long *counters) {
    extern __shared__ __align__(16) unsigned char lsm[];
    const int64_t cnt = (int64_t)counters[C_ORD_LEN];
    constexpr int PW = 64 / G;
    if ((int64_t)blockIdx.x * (LP_THREADS / G) >= cnt) return;  // whole blocks, before any barrier
    LpNeighbour *nb = reinterpret_cast<LpNeighbour *>(lsm) + (threadIdx.x & ~(G - 1));
    unsigned short *pairs = reinterpret_cast<unsigned short *>(reinterpret_cast<LpNeighbour *>(lsm) + LP_THREADS);
    lp_pairs(pairs, e.use_cutoff ? e.k - 1 : e.k);
    const int64_t wave = (int64_t)blockIdx.x * (LP_THREADS / 64) + (threadIdx.x >> 6);
    const int64_t nw = (int64_t)gridDim.x * (LP_THREADS / 64);
    for (int64_t p0 = wave * PW; p0 < cnt; p0 += nw * PW) {
        const int64_t at = p0 + (threadIdx.x & 63) / G;
        const bool on = at < cnt;
        lp_point<G, 2>(e, on ? (int64_t)list[cap - 1 - at] : 0, on, nb, pairs);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        atomicAdd(&counters[C_FALLBACK], (unsigned long long)cnt);
        atomicAdd(&counters[C_NEARTIE], (unsigned long long)cnt);
    }
}

hipError_t launch_reorder(const EmbedArgs &a, int num_cus, hipStream_t s) {
    ListArgs e;
    memset(&e, 0, sizeof e);
    e.X = a.X;
    e.n = a.n;
    e.ldx = a.ldx;
    e.d = a.d;
    e.dp = a.dp;
    e.g = a.g;
    e.k = a.k;
    e.use_cutoff = a.use_cutoff;
    e.Lpad = a.Lpad;
    e.ipos = a.ipos;
    e.l = a.l2d;
    e.knn_idx = a.knn_idx;
    for (int i = 1; i <= a.k; ++i) e.Wk += 1.0 / i;
    e.boost = a.boost;
    e.cutoff = a.cutoff;
    e.gravity = a.gravity;
    e.adjust = a.adjust;
    e.out = a.out;
    e.out_idx = a.knn_idx;
    e.out_d2 = a.knn_d2;
    // the list's length is only known on the device: a fixed grid loops over it
    const int gl = a.k <= 16 ? 16 : a.k <= 32 ? 32 : 64;
    auto kern = gl == 16 ? embed_reorder<16> : gl == 32 ? embed_reorder<32> : embed_reorder<64>;
    const long long per = LP_THREADS / gl;
    long long blocks = (a.n + per - 1) / per;
    if (blocks > (long long)num_cus * 8) blocks = (long long)num_cus * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(LP_THREADS), lp_lds_bytes(a.k), s, e, a.fb_list, a.fb_cap,
                       a.counters);
    return hipGetLastError();
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
