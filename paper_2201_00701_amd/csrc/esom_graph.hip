// Graph-mode supervision (Section "Semi-supervised structure reconstruction"):
// the neighbourhood graph of the high-dimensional landmarks, a force-based
// layout of their 2-D positions on that graph, and the duplication and
// removal of landmarks.  The paper names no graph or force law; the graph is
// the kg nearest other landmarks of every landmark and the force law is a
// spring per edge (rest length proportional to the high-dimensional distance)
// plus a softened all-pairs repulsion.
#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "esom_internal.h"

namespace esom {

// Wavefront minima (device library, DPP reductions).
extern "C" __device__ double __ockl_wfred_min_f64(double);
extern "C" __device__ int __ockl_wfred_min_i32(int);

// Lexicographic order on (squared distance, index).
__device__ __forceinline__ bool pair_before(double da, int ia, double db, int ib) {
    return da < db || (da == db && ia < ib);
}

// Neighbourhood graph: GRAPH_U landmarks u per block, each with VG wavefronts.
// The block stages tiles of 64 VG landmark rows in LDS (row stride odd: no bank
// conflicts between the lanes' rows); lane i of wavefront (u, vg) takes row
// 64 vg + i of every tile and keeps its KC nearest in a sorted register list
// (KC = 8, 16 or 32: the smallest that holds kg).  The wavefront merges its 64
// lists by kg rounds of a wave minimum, and the VG lists of a landmark are
// merged by counting ranks.  Distances are FP64 sums of squared differences,
// added in dimension order without fused multiply-adds, so equal distances
// compare equal exactly as in a plain double-precision evaluation.
// Bound by the latency of the serial FP64 sums and insertions, so VG = 4 where
// the tile fits (up to 128 dimensions), 1 above.  1024 landmarks of 48
// dimensions, kg = 10: 121 us with one wavefront per landmark that read the
// rows from memory lane by lane (64 lines a load) into a 32-slot list; 63 us
// with staged tiles and VG = 1; 36 us with VG = 4.
constexpr int GRAPH_U = 4;
constexpr int GRAPH_VG = 4;
constexpr int GRAPH_VG_MAX_D = 128;

__host__ __device__ inline int graph_row_stride(int d) { return d | 1; }

template <int KC>
__global__ void __launch_bounds__(64 * GRAPH_U * GRAPH_VG) landmark_graph_kernel(const float *__restrict__ L, int g,
                                                                                 int d, int kg,
                                                                                 int32_t *__restrict__ nbr,
                                                                                 float *__restrict__ dist2) {
    extern __shared__ __align__(16) unsigned char gsm[];
    __shared__ double ld[GRAPH_U][GRAPH_VG * KC];  // the wavefronts' merged lists
    __shared__ int li[GRAPH_U][GRAPH_VG * KC];
    double *own = reinterpret_cast<double *>(gsm);              // GRAPH_U x d: the rows of the block's landmarks
    float *tile = reinterpret_cast<float *>(own + GRAPH_U * d);  // 64 VG rows
    const int rs = graph_row_stride(d);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int VG = blockDim.x / (64 * GRAPH_U);
    const int uu = wv / VG, vg = wv % VG;
    const int u0 = blockIdx.x * GRAPH_U, u = u0 + uu;
    for (int e = threadIdx.x; e < GRAPH_U * d; e += blockDim.x)
        own[e] = u0 * d + e < g * d ? (double)L[u0 * d + e] : 0.0;
    double bd[KC];
    int bi[KC];
#pragma unroll
    for (int q = 0; q < KC; ++q) {
        bd[q] = INFINITY;
        bi[q] = INT32_MAX;
    }
    const double *Lu = own + uu * d;
    const int nt = blockDim.x, step_r = nt / d, step_t = nt % d;
    for (int v0 = 0; v0 < g; v0 += 64 * VG) {
        __syncthreads();
        // the tile's rows are contiguous in L; 8 loads of a thread in flight
        const int cnt = (g - v0 < 64 * VG ? g - v0 : 64 * VG) * d;
        const float *Lt = L + (size_t)v0 * d;
        int r = (int)threadIdx.x / d, t = (int)threadIdx.x % d;
        for (int e0 = threadIdx.x; e0 < cnt; e0 += 8 * nt) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = e0 + i * nt < cnt ? Lt[e0 + i * nt] : 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (e0 + i * nt < cnt) tile[r * rs + t] = x[i];
                r += step_r;
                t += step_t;
                if (t >= d) {
                    t -= d;
                    ++r;
                }
            }
        }
        __syncthreads();
        const int v = v0 + 64 * vg + lane;
        const bool live = v < g && v != u;
        const float *Lv = tile + (live ? 64 * vg + lane : 0) * rs;
        double s = 0.0;
#pragma unroll 8
        for (int q = 0; q < d; ++q) {
            const double df = (double)Lv[q] - Lu[q];
            s = __dadd_rn(s, __dmul_rn(df, df));
        }
        // an infinite distance (no finite one reaches DBL_MAX) competes by index
        const double cd = !live ? INFINITY : s == INFINITY ? DBL_MAX : s;
        if (__ballot(cd < bd[KC - 1]) == 0ull) continue;
        // v ascends, so a tie keeps the earlier entry first and a strict
        // comparison orders by (distance, index); every slot after the
        // insertion takes its predecessor
#pragma unroll
        for (int q = KC - 1; q >= 0; --q) {
            const bool here = cd < bd[q];
            const bool shift = q > 0 && cd < bd[q > 0 ? q - 1 : 0];
            bd[q] = shift ? bd[q > 0 ? q - 1 : 0] : here ? cd : bd[q];
            bi[q] = shift ? bi[q > 0 ? q - 1 : 0] : here ? v : bi[q];
        }
    }
    // kg rounds, each taking the wave-wide smallest head by (distance, index)
    for (int r = 0; r < kg; ++r) {
        const double md = __ockl_wfred_min_f64(bd[0]);
        const int mi = __ockl_wfred_min_i32(bd[0] == md ? bi[0] : INT32_MAX);
        if (lane == 0) {
            ld[uu][vg * kg + r] = md;
            li[uu][vg * kg + r] = mi;
        }
        // the lane whose head was taken pops it (indices are unique)
        if (bi[0] == mi && mi < g) {
#pragma unroll
            for (int q = 0; q + 1 < KC; ++q) {
                bd[q] = bd[q + 1];
                bi[q] = bi[q + 1];
            }
            bd[KC - 1] = INFINITY;
            bi[KC - 1] = INT32_MAX;
        }
    }
    __syncthreads();
    if (vg != 0 || u >= g) return;
    // ranks by (distance, index); empty entries (+inf, INT32_MAX) by their place
    for (int c = lane; c < VG * kg; c += 64) {
        const double dc = ld[uu][c];
        const int jc = li[uu][c];
        int rank = 0;
        for (int o = 0; o < VG * kg; ++o) {
            const double dd = ld[uu][o];
            const int jo = li[uu][o];
            rank += (pair_before(dd, jo, dc, jc) || (dd == dc && jo == jc && o < c)) ? 1 : 0;
        }
        if (rank < kg) {
            nbr[(size_t)u * kg + rank] = jc < g ? jc : -1;
            if (dist2) dist2[(size_t)u * kg + rank] = jc < g ? (float)dc : INFINITY;
        }
    }
}

hipError_t launch_landmark_graph(const float *L, int g, int d, int kg, int32_t *nbr, float *dist2,
                                 hipStream_t s) {
    const unsigned blocks = (unsigned)((g + GRAPH_U - 1) / GRAPH_U);
    const int vg = d <= GRAPH_VG_MAX_D ? GRAPH_VG : 1;
    const size_t smem = sizeof(double) * GRAPH_U * d + sizeof(float) * 64 * vg * graph_row_stride(d);
    auto kern = kg <= 8 ? landmark_graph_kernel<8> : kg <= 16 ? landmark_graph_kernel<16> : landmark_graph_kernel<32>;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * GRAPH_U * vg), smem, s, L, g, d, kg, nbr, dist2);
    return hipGetLastError();
}

// ---------------------------------------------------------------- layout
// A layout call first turns the neighbour lists into each node's own edge list
// (layout_edges, once per call: the graph does not change between the steps),
// then runs its steps, one wavefront per node: the lanes share the all-pairs
// repulsion and the node's edges, forces and the move are summed in FP64 from
// the positions before the step (lin), and the new positions go to lout.
// The steps used to give a node one thread, which searched every other node's
// neighbour list in every step: at g = 1024, kg = 10 four blocks took 3109 us a
// step; now 6 us a step and 23 us for the lists, most of it the
// launches.
constexpr int LAYOUT_THREADS = 256;
constexpr int LAYOUT_WORDS = (ESOM_MAX_G + 31) / 32;  // bitmap words of a node's partners
static_assert(LAYOUT_WORDS <= LAYOUT_THREADS, "one bitmap word per thread");

// The partners of node u in the undirected graph (v in u's list or u in v's
// list, v != u) as a bitmap in LDS: bit v of mask.  All threads of the block;
// ends with a barrier.
__device__ __forceinline__ void layout_partners(const int32_t *__restrict__ nbr, int g, int kg, int u,
                                                unsigned *mask) {
    for (int w = threadIdx.x; w < LAYOUT_WORDS; w += blockDim.x) mask[w] = 0u;
    __syncthreads();
    for (int q = threadIdx.x; q < kg; q += blockDim.x) {
        const int v = nbr[(size_t)u * kg + q];
        if (v >= 0 && v < g && v != u) atomicOr(&mask[v >> 5], 1u << (v & 31));
    }
    for (int e0 = threadIdx.x; e0 < g * kg; e0 += 8 * LAYOUT_THREADS) {
        int x[8];  // 8 loads in flight
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = e0 + i * LAYOUT_THREADS < g * kg ? nbr[e0 + i * LAYOUT_THREADS] : -1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (x[i] == u) {
                const int v = (e0 + i * LAYOUT_THREADS) / kg;
                if (v != u) atomicOr(&mask[v >> 5], 1u << (v & 31));
            }
        }
    }
    __syncthreads();
}

__device__ __forceinline__ double layout_rest(const float *__restrict__ L, int d, int u, int v) {
    const float *Lu = L + (size_t)u * d, *Lv = L + (size_t)v * d;
    double hd = 0.0;
#pragma unroll 8
    for (int t = 0; t < d; ++t) {
        const double df = (double)Lu[t] - (double)Lv[t];
        hd = fma(df, df, hd);
    }
    return sqrt(hd);
}

__global__ void layout_zero(unsigned *cursor) {
    if (threadIdx.x == 0) *cursor = 0u;
}

// Edge list of node u = blockIdx.x, partners ascending with their distances
// |L_u - L_v|: span[u] = (first entry, count).  Each listed neighbour makes at
// most two entries, so 2 g kg entries hold them all; the blocks claim their
// ranges from the cursor (their order in the array has no effect).
__global__ void __launch_bounds__(LAYOUT_THREADS) layout_edges(const float *__restrict__ L, int g, int d,
                                                               const int32_t *__restrict__ nbr, int kg,
                                                               unsigned *cursor, uint2 *__restrict__ span,
                                                               LayoutEdge *__restrict__ edges) {
    __shared__ unsigned mask[LAYOUT_WORDS];
    __shared__ unsigned wsum[LAYOUT_THREADS / 64], base;
    __shared__ unsigned short list[ESOM_MAX_G];
    const int u = blockIdx.x;
    layout_partners(nbr, g, kg, u, mask);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    unsigned w = (int)threadIdx.x < LAYOUT_WORDS ? mask[threadIdx.x] : 0u;
    const unsigned c = __popc(w);
    unsigned incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    unsigned at = incl - c, total = 0;
#pragma unroll
    for (int q = 0; q < LAYOUT_THREADS / 64; ++q) {
        at += q < wv ? wsum[q] : 0u;
        total += wsum[q];
    }
    for (; w; w &= w - 1u) list[at++] = (unsigned short)(32 * threadIdx.x + __ffs(w) - 1);
    if (threadIdx.x == 0) {
        base = atomicAdd(cursor, total);
        span[u] = make_uint2(base, total);
    }
    __syncthreads();
    for (unsigned i = threadIdx.x; i < total; i += blockDim.x) {
        LayoutEdge ed;
        ed.v = list[i];
        ed.rest = layout_rest(L, d, u, ed.v);
        edges[base + i] = ed;
    }
}

// Repulsion of all other nodes on one at (ux, uy), summed by the calling
// wavefront's lanes (the node's own term is 0: no difference).
__device__ __forceinline__ void layout_repel(const float *__restrict__ lin, int g, int lane, double ux, double uy,
                                             double repulsion, double soft2, double &fx, double &fy) {
    for (int v = lane; v < g; v += 64) {
        const float2 pv = reinterpret_cast<const float2 *>(lin)[v];
        const double dx = (double)pv.x - ux, dy = (double)pv.y - uy;
        const double push = repulsion / (dx * dx + dy * dy + soft2);
        fx = fma(-push, dx, fx);
        fy = fma(-push, dy, fy);
    }
}

// Spring of an edge to the node at pv with rest length `rest` (none while the
// two coincide).
__device__ __forceinline__ void layout_pull(float2 pv, double ux, double uy, double rest, double &fx, double &fy) {
    const double dx = (double)pv.x - ux, dy = (double)pv.y - uy;
    const double r = sqrt(dx * dx + dy * dy);
    if (r > 0.0) {
        const double pull = (r - rest) / r;
        fx = fma(pull, dx, fx);
        fy = fma(pull, dy, fy);
    }
}

__device__ __forceinline__ double layout_wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ void layout_move(float *__restrict__ lout, const uint8_t *__restrict__ fixed, int u,
                                            double ux, double uy, double fx, double fy, double step,
                                            double max_move) {
    double mx = step * fx, my = step * fy;
    const double len = sqrt(mx * mx + my * my);
    if (len > max_move) {
        mx *= max_move / len;
        my *= max_move / len;
    }
    if (fixed && fixed[u]) mx = my = 0.0;
    reinterpret_cast<float2 *>(lout)[u] = make_float2((float)(ux + mx), (float)(uy + my));
}

// One synchronous step from the edge lists, one wavefront per node.
__global__ void __launch_bounds__(LAYOUT_THREADS) layout_step_kernel(
    int g, const uint2 *__restrict__ span, const LayoutEdge *__restrict__ edges, const float *__restrict__ lin,
    float *__restrict__ lout, const uint8_t *__restrict__ fixed, double scale, double repulsion, double soft2,
    double step, double max_move) {
    const int lane = threadIdx.x & 63;
    const int u = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    if (u >= g) return;  // whole wavefronts
    const float2 pu = reinterpret_cast<const float2 *>(lin)[u];
    const uint2 sp = span[u];
    const double ux = pu.x, uy = pu.y;
    double fx = 0.0, fy = 0.0;
    for (unsigned i = lane; i < sp.y; i += 64) {
        const LayoutEdge ed = edges[sp.x + i];
        layout_pull(reinterpret_cast<const float2 *>(lin)[ed.v], ux, uy, scale * ed.rest, fx, fy);
    }
    layout_repel(lin, g, lane, ux, uy, repulsion, soft2, fx, fy);
    fx = layout_wave_sum(fx);
    fy = layout_wave_sum(fy);
    if (lane == 0) layout_move(lout, fixed, u, ux, uy, fx, fy, step, max_move);
}

// The same step without edge lists, for a context whose memory budget has no
// room for them: one block per node finds the node's partners itself.
__global__ void __launch_bounds__(LAYOUT_THREADS) layout_step_search(
    const float *__restrict__ L, int g, int d, const int32_t *__restrict__ nbr, int kg,
    const float *__restrict__ lin, float *__restrict__ lout, const uint8_t *__restrict__ fixed, double scale,
    double repulsion, double soft2, double step, double max_move) {
    __shared__ unsigned mask[LAYOUT_WORDS];
    const int u = blockIdx.x;
    layout_partners(nbr, g, kg, u, mask);
    if (threadIdx.x >= 64) return;  // the first wavefront sums
    const int lane = threadIdx.x;
    const float2 pu = reinterpret_cast<const float2 *>(lin)[u];
    const double ux = pu.x, uy = pu.y;
    double fx = 0.0, fy = 0.0;
    for (int v = lane; v < g; v += 64)
        if ((mask[v >> 5] >> (v & 31)) & 1u)
            layout_pull(reinterpret_cast<const float2 *>(lin)[v], ux, uy, scale * layout_rest(L, d, u, v), fx, fy);
    layout_repel(lin, g, lane, ux, uy, repulsion, soft2, fx, fy);
    fx = layout_wave_sum(fx);
    fy = layout_wave_sum(fy);
    if (lane == 0) layout_move(lout, fixed, u, ux, uy, fx, fy, step, max_move);
}

// Workspace of a layout call: the other position buffer, then (edges != 0) the
// cursor, the spans and the edge lists for the largest kg, so that its size
// depends on g alone.
size_t layout_workspace_bytes(int g, int edges) {
    size_t b = (sizeof(float) * 2 * (size_t)g + 255) & ~(size_t)255;
    if (edges) b += 256 + ((sizeof(uint2) * (size_t)g + 255) & ~(size_t)255) +
                    sizeof(LayoutEdge) * 2 * (size_t)g * GRAPH_MAX_K;
    return b;
}

hipError_t launch_layout(const float *L, int g, int d, const int32_t *nbr, int kg, float *l2d, void *ws, int edges,
                         const uint8_t *fixed, int steps, double scale, double repulsion, double soft, double step,
                         double max_move, hipStream_t s) {
    char *p = static_cast<char *>(ws);
    float *other = reinterpret_cast<float *>(p);
    p += (sizeof(float) * 2 * (size_t)g + 255) & ~(size_t)255;
    unsigned *cursor = reinterpret_cast<unsigned *>(p);
    p += 256;
    uint2 *span = reinterpret_cast<uint2 *>(p);
    p += (sizeof(uint2) * (size_t)g + 255) & ~(size_t)255;
    LayoutEdge *ed = reinterpret_cast<LayoutEdge *>(p);
    if (edges) {
        hipLaunchKernelGGL(layout_zero, dim3(1), dim3(64), 0, s, cursor);
        hipLaunchKernelGGL(layout_edges, dim3(g), dim3(LAYOUT_THREADS), 0, s, L, g, d, nbr, kg, cursor, span, ed);
    }
    // synchronous steps alternate between l2d and the workspace; an odd count
    // ends in the workspace and is copied back
    float *bufs[2] = {l2d, other};
    for (int t = 0; t < steps; ++t) {
        if (edges)
            hipLaunchKernelGGL(layout_step_kernel, dim3((g + LAYOUT_THREADS / 64 - 1) / (LAYOUT_THREADS / 64)),
                               dim3(LAYOUT_THREADS), 0, s, g, span, ed, bufs[t & 1], bufs[(t + 1) & 1], fixed, scale,
                               repulsion, soft * soft, step, max_move);
        else
            hipLaunchKernelGGL(layout_step_search, dim3(g), dim3(LAYOUT_THREADS), 0, s, L, g, d, nbr, kg,
                               bufs[t & 1], bufs[(t + 1) & 1], fixed, scale, repulsion, soft * soft, step, max_move);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && (steps & 1))
        e = hipMemcpyAsync(l2d, other, sizeof(float) * 2 * (size_t)g, hipMemcpyDeviceToDevice, s);
    return e;
}

// Landmark g (a new row) := landmark j, 2-D position shifted by (dx, dy).
__global__ void duplicate_kernel(float *__restrict__ L, float *__restrict__ l2d, int g, int d, int j, float dx,
                                 float dy) {
    for (int t = threadIdx.x; t < d; t += blockDim.x) L[(size_t)g * d + t] = L[(size_t)j * d + t];
    if (threadIdx.x == 0) {
        l2d[2 * g] = l2d[2 * j] + dx;
        l2d[2 * g + 1] = l2d[2 * j + 1] + dy;
    }
}

// Landmark j := landmark g - 1 (the last row moves into the removed slot).
__global__ void remove_kernel(float *__restrict__ L, float *__restrict__ l2d, int g, int d, int j) {
    const int last = g - 1;
    for (int t = threadIdx.x; t < d; t += blockDim.x) L[(size_t)j * d + t] = L[(size_t)last * d + t];
    if (threadIdx.x == 0) {
        l2d[2 * j] = l2d[2 * last];
        l2d[2 * j + 1] = l2d[2 * last + 1];
    }
}

hipError_t launch_duplicate(float *L, float *l2d, int g, int d, int j, float dx, float dy, hipStream_t s) {
    hipLaunchKernelGGL(duplicate_kernel, dim3(1), dim3(256), 0, s, L, l2d, g, d, j, dx, dy);
    return hipGetLastError();
}

hipError_t launch_remove(float *L, float *l2d, int g, int d, int j, hipStream_t s) {
    hipLaunchKernelGGL(remove_kernel, dim3(1), dim3(256), 0, s, L, l2d, g, d, j);
    return hipGetLastError();
}

}  // namespace esom
