// Fused EmbedSOM kernel for gfx950 (one wavefront = 64 points).
//
// Phase A, screen (MFMA).  The wave holds its 64 points as two 32-point MFMA
// B operands (centred on the landmark centroid) in registers and streams
// 32-landmark A tiles (-2 (L_j - c), prepared once per landmark set).
// v_mfma_f32_32x32x* with C initialised to |L_j - c|^2 gives
//   key_ij = |L_j - c|^2 - 2 <x_i - c, L_j - c>  =  delta_ij^2 - |x_i - c|^2,
// so keys rank the landmarks of a point exactly like the distances do.  In
// the 32x32 output layout lane l holds 16 keys of point (l mod 32); the two
// lanes l and l+32 of a point see disjoint halves of every tile.
//   Pass 1 (BF16 operands) keeps, per lane, the minimum key of 32 landmark
//   groups (register slot x tile parity).  The C-th smallest of a point's 64
//   group minima bounds from above C distinct keys; widened by both passes'
//   error bounds it is the threshold tau.  Points in locality order also keep
//   each tile's minimum, and pass 2 leaves out the tiles that lie above tau.
//   Pass 2 recomputes the keys more accurately (FP32 operands in FP32 mode;
//   in BF16 mode both operands split into high and low BF16 parts, three
//   products per element, which leaves an error near 2^-16 of the products
//   instead of 2^-8) and shifts one bit per key (key <= tau) into a per-lane
//   bitmap in LDS: the candidate set, with no capacity limit.
// Phase B, exact selection (one lane = one point; rows streamed from L2 are read
// by quads of lanes).  Every candidate is
// rescored with exact FP32 differences and inserted into a sorted register
// list; keys are doubles packing (delta^2, landmark index) so a plain
// min/max network orders them lexicographically.  A point is certified when
// its k-th rescored distance lies below tau by more than a rigorous bound of
// the screen's rounding error (every non-candidate then lies farther away).
// Phase C, projection (FP32, FP64 solve).  Scores from the k distances; the
// pair terms use D_uv = 1/2 + (delta_u^2 - delta_v^2) / (2 |L_u - L_v|^2)
// (polarisation of the segment projection) with the pair table from the
// landmark preparation; Cramer's rule in FP64.
// Points the fast path cannot vouch for (uncertified screen, k-th/(k+1)-th
// tie below FP32 resolution, ill-conditioned system, degenerate
// neighbourhood) are appended to a list and recomputed by the exact FP64
// kernel afterwards.
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "esom_internal.h"

namespace esom {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr float U32 = 5.9604645e-08f;     // 2^-24, FP32 unit roundoff
constexpr float ILL_PAIR = 64.0f;         // max(delta^2)/(2|L_u-L_v|^2) beyond this: exact path
constexpr double ILL_COND = 64.0;         // (tr/2)^2/det beyond this: exact path
constexpr double SINGULAR_REL = 1e-9;     // det <= this (tr/2)^2: singular, centroid
// Cutoff weights below this are recomputed from FP64 distances: c = 1 - exp(A
// (delta_q - delta_k) / delta_k) takes its relative accuracy from the difference
// delta_q - delta_k, which FP32 distances only give to ~u delta_k, so a weight
// c ~ A u carries a relative error near 1 (and a system held only by such a
// weight moves accordingly).  Above it the relative error is at most
// 2 A (d_pad + 3) u / C_REFINE.  Done for k <= 8 (see embed_main).
constexpr float C_REFINE = 1.0f / 32.0f;
constexpr float LN_1M_CREFINE = -0.031748698f;  // ln(1 - C_REFINE)
constexpr int N_REFINE = 4;                      // refined weights per point at most

// Largest block of the fused kernel: 12 waves (3 per SIMD, 168 registers per
// lane) where the register budget of the instantiation allows it (padded
// dimension <= 32, k <= 16), else 8 waves (256 registers).  In FP32 mode the
// 12-wave block leaves no LDS room for the FP32 screen tiles (they stream
// from L2) and spills a few registers once per 64 points, and still runs
// 8% faster at 1M x 32-D with 400 landmarks than 8 waves with the tiles in
// LDS: the third wave per SIMD overlaps one wave's MFMA screen with another's
// VALU phases.
__host__ __device__ constexpr int main_max_block(int mode, int dc, int kp) {
    return (dc <= 2 && kp <= 16) ? 768 : 512;
}

// 1 - exp(z) for z <= 0 with full relative accuracy near 0: Taylor series
// through z^7 for |z| < 1/8 (truncation below 2e-11 relative), else 1 - exp(z)
// directly (then 1 - exp(z) > 0.11 and its rounding is relatively small).
__device__ __forceinline__ float one_minus_exp(float z) {
    if (z > -0.125f) {
        float p = 1.f / 5040.f;
        p = fmaf(p, z, 1.f / 720.f);
        p = fmaf(p, z, 1.f / 120.f);
        p = fmaf(p, z, 1.f / 24.f);
        p = fmaf(p, z, 1.f / 6.f);
        p = fmaf(p, z, 0.5f);
        p = fmaf(p, z, 1.f);
        return fmaxf(-z * p, 0.f);
    }
    return 1.f - __expf(z);
}

__device__ __forceinline__ unsigned bf16_bits_rne(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// Two floats rounded to BF16 (to nearest even), the first in the low half.
__device__ __forceinline__ unsigned bf16_pair(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ double pack_key(float d2, int j) {
    unsigned long long b = (unsigned long long)__double_as_longlong((double)d2);
    return __longlong_as_double((long long)(b | (unsigned long long)j));
}
__device__ __forceinline__ float key_d2(double v) {
    unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (float)__longlong_as_double((long long)(b & ~0x1FFFull));
}
__device__ __forceinline__ int key_idx(double v) {
    return (int)((unsigned long long)__double_as_longlong(v) & 0x1FFFull);
}

// Upper bound of the exact k-th nearest squared distance from the rescored
// k-th value d2k: each of the first k rescored values is within (d_pad+3)u of
// its exact value, so k landmarks lie within d2k (1 + 2 (d_pad+3) u); the
// factor 4 leaves room for the FP64 distances of the exact path.  +inf when
// fewer than k candidates were rescored (d2k = +inf).
__device__ __forceinline__ float kth_bound(float d2k, int dp) {
    const float t = d2k * (1.f + 4.f * (float)(dp + 3) * U32);
    return t < FLT_MAX ? t : INFINITY;
}

// Batcher's odd-even merge sort network on N = 2^m inputs (63 comparators for
// 16, 191 for 32), built at compile time.
template <int N>
struct OemNet {
    int a[N * N] = {}, b[N * N] = {};
    int n = 0;
    constexpr OemNet() { sort(0, N - 1); }
    constexpr void merge(int lo, int hi, int r) {
        const int step = 2 * r;
        if (step < hi - lo) {
            merge(lo, hi, step);
            merge(lo + r, hi, step);
            for (int i = lo + r; i < hi - r; i += step) {
                a[n] = i;
                b[n] = i + r;
                ++n;
            }
        } else {
            a[n] = lo;
            b[n] = lo + r;
            ++n;
        }
    }
    constexpr void sort(int lo, int hi) {
        if (hi - lo >= 1) {
            const int mid = lo + (hi - lo) / 2;
            sort(lo, mid);
            sort(mid + 1, hi);
            merge(lo, hi, 1);
        }
    }
};

// Ascending sort of N registers.  The screen sorts bit patterns of
// non-negative floats: for those, integer order is float order and +inf sorts
// last.
template <int N>
__device__ __forceinline__ void sort_regs(int (&v)[N]) {
    constexpr OemNet<N> net{};
#pragma unroll
    for (int c = 0; c < net.n; ++c) {
        const int x = v[net.a[c]], y = v[net.b[c]];
        v[net.a[c]] = min(x, y);
        v[net.b[c]] = max(x, y);
    }
}

// Bitonic merge of N registers holding a bitonic sequence: ascending after.
template <int N>
__device__ __forceinline__ void bitonic_clean(int (&m)[N]) {
#pragma unroll
    for (int st = N / 2; st > 0; st >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((i & st) == 0) {
                const int x = m[i], y = m[i + st];
                m[i] = min(x, y);
                m[i + st] = max(x, y);
            }
}

// The j-th smallest (1 <= j <= 32) of the 64 values held by a lane (lo[0..15],
// hi[0..15]) and its partner lane (lane ^ 32), the same on both lanes.  Each
// lane orders its own smallest values (16 for j <= 16, else all 32); with two
// ascending lists s and t of length M, min(s[i], t[M - 1 - i]) holds the M
// smallest of their union as a bitonic sequence, which a bitonic merge orders.
// j is uniform.
__device__ __forceinline__ int select_pair_jth(int (&lo)[16], int (&hi)[16], int j) {
    if (j <= 16) {
        sort_regs<16>(lo);
        sort_regs<16>(hi);
        int s[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = min(lo[i], hi[15 - i]);
        bitonic_clean<16>(s);
        int u[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) u[i] = min(s[i], __shfl_xor(s[15 - i], 32));
        bitonic_clean<16>(u);
        int t = u[0];
#pragma unroll
        for (int i = 1; i < 16; ++i)
            if (i == j - 1) t = u[i];
        return t;
    }
    int v[32];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        v[i] = lo[i];
        v[16 + i] = hi[i];
    }
    sort_regs<32>(v);
    int u[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) u[i] = min(v[i], __shfl_xor(v[31 - i], 32));
    bitonic_clean<32>(u);
    int t = u[31];
#pragma unroll
    for (int i = 16; i < 31; ++i)
        if (i == j - 1) t = u[i];
    return t;
}

// An upper bound of the J-th smallest (compile-time, 8 <= J <= 24) of those 64
// values, the same on both lanes: the J-th smallest of the two lanes' M smallest
// (M = 8 or 16), which is the J-th of all unless one lane holds more than M of
// them (possible for J > M only).  With two ascending lists s and t the J-th
// smallest of their union is the minimum over a + b = J of max(s_a, t_b) (s_0 =
// t_0 = -inf), so the two lanes' lists need no merge.  About 400 instructions
// for J = 16 and 20 where select_pair_jth takes 460 and 820 (1M x 48-D, k = 20:
// with the conversion instructions for the operands, fused kernel 0.790 ->
// 0.744 ms; 10M x 64-D 8.4 -> 7.85 ms).
template <int J>
__device__ __forceinline__ int select_pair_static(int (&lo)[16], int (&hi)[16]) {
    constexpr int M = J <= 8 ? 8 : 16;
    static_assert(J <= 24 && J <= 2 * M, "list length");
    sort_regs<16>(lo);
    sort_regs<16>(hi);
    int s[M];
#pragma unroll
    for (int i = 0; i < M; ++i) s[i] = min(lo[i], hi[M - 1 - i]);
    bitonic_clean<M>(s);
    int u[M], v[M];  // the lower and the upper lane's lists, on both
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap((unsigned)s[i], (unsigned)s[i], false, false);
        u[i] = (int)r[0];
        v[i] = (int)r[1];
    }
    int t = 0x7FFFFFFF;
#pragma unroll
    for (int i = 0; i <= M; ++i) {  // i values of the first list, J - i of the second
        if (J - i < 0 || J - i > M) continue;
        const int x = i == 0 ? v[J - 1] : J - i == 0 ? u[i - 1] : max(u[i > 0 ? i - 1 : 0], v[J - i > 0 ? J - i - 1 : 0]);
        t = min(t, x);
    }
    return t;
}

// The j-th smallest (1 <= j <= 32) of the 32 values lo[0..15], hi[0..15].
// For j <= 16: with both halves sorted, min(lo[i], hi[15 - i]) holds the 16
// smallest of the union as a bitonic sequence; its maximum is the 16th
// smallest, and a bitonic merge orders it for smaller j.  j is uniform.
__device__ __forceinline__ int select_jth(int (&lo)[16], int (&hi)[16], int j) {
    if (j <= 16) {
        sort_regs<16>(lo);
        sort_regs<16>(hi);
        int m[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) m[i] = min(lo[i], hi[15 - i]);
        if (j == 16) {
            int t = m[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) t = max(t, m[i]);
            return t;
        }
#pragma unroll
        for (int st = 8; st > 0; st >>= 1)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((i & st) == 0) {
                    const int x = m[i], y = m[i + st];
                    m[i] = min(x, y);
                    m[i + st] = max(x, y);
                }
        int t = m[0];
#pragma unroll
        for (int i = 1; i < 16; ++i)
            if (i == j - 1) t = m[i];
        return t;
    }
    int v[32];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        v[i] = lo[i];
        v[16 + i] = hi[i];
    }
    sort_regs<32>(v);
    int t = v[31];
#pragma unroll
    for (int i = 16; i < 32; ++i)
        if (i == j - 1) t = v[i];
    return t;
}

// FP32 minimum as a single instruction: the median of (a, b, ninf) with ninf
// = -inf.  fminf, or a median with a visible -inf constant (which the
// compiler turns into fminf), quiets both operands with an extra instruction
// each.  (Not inline assembly: the compiler must see the read of an MFMA
// result to insert the wait states it needs.)
__device__ __forceinline__ float vmin32(float a, float b, float ninf) {
    return __builtin_amdgcn_fmed3f(a, b, ninf);
}

// x * y as a 24-bit multiply (full rate); the compiler otherwise emits a
// 32-bit multiply, which issues at a quarter of the rate.  x, y < 2^24 and
// x * y < 2^32.
__device__ __forceinline__ unsigned mul24(unsigned x, unsigned y) {
    unsigned r;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(x), "s"(y));
    return r;
}
template <int RS>
__device__ __forceinline__ unsigned row_offset(int j) {
    return mul24((unsigned)j, (unsigned)RS);
}

// Orders this wavefront's LDS accesses before and after it (its lanes exchange
// data through LDS; the hardware keeps a wavefront's LDS accesses in order).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// -inf in a scalar register, opaque to the compiler.
__device__ __forceinline__ float opaque_neg_inf() {
    float r;
    asm volatile("s_mov_b32 %0, 0xff800000" : "=s"(r));
    return r;
}

// FP64 minimum / maximum as single instructions.  fmin/fmax would add a
// quieting step per operand for signalling NaNs, which never occur here (the
// operands are packed keys of finite distances, or +inf).
__device__ __forceinline__ double vmin64(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double vmax64(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The value of lane S of the calling lane's quad, and the sum over a quad (the
// same on its four lanes).  All lanes of the wavefront take part.
template <int S>
__device__ __forceinline__ int quad_bcast(int v) {
    return __builtin_amdgcn_mov_dpp(v, S * 0x55, 0xf, 0xf, true);
}
__device__ __forceinline__ float quad_sum(float v) {
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true));  // lanes 1 0 3 2
    v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true));  // lanes 2 3 0 1
    return v;
}
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double quad_sum64(double v) {
    v += dpp64<0xB1>(v);
    v += dpp64<0x4E>(v);
    return v;
}

// The value of lane U of the calling lane's row of 16 lanes.
template <int U>
__device__ __forceinline__ unsigned row16_bcast(unsigned v) {
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x150 + U, 0xf, 0xf, true);
}

// f(IntTag<A>{}), ..., f(IntTag<B - 1>{})
template <int A, int B, class F>
__device__ __forceinline__ void static_for(F &&f);

// Insert v into the ascending list s; whatever falls off the end updates rej
// (the smallest key ever rejected).  Every slot becomes min(s[q], max(s[q - 1],
// v)) of the old values, from the end on in place: the same two operations a slot
// as carrying the displaced value along, without its chain of KP maxima.
template <int KP>
__device__ __forceinline__ void insert_sorted(double (&s)[KP], double &rej, double v) {
    rej = vmin64(rej, vmax64(s[KP - 1], v));
#pragma unroll
    for (int q = KP - 1; q > 0; --q) {
        const double t = vmax64(s[q - 1], v);
        asm("v_min_f64 %0, %0, %1" : "+v"(s[q]) : "v"(t));  // in place: no copies of the list
    }
    asm("v_min_f64 %0, %0, %1" : "+v"(s[0]) : "v"(v));
}

// Next non-empty 64-bit bitmap word of a point: mk marks the non-empty words
// (bit tp = tile pair tp), row = the point's words, stride 32 per tile pair.
// nb = 0 when none is left.
__device__ __forceinline__ void next_word(unsigned long long &mk, const unsigned long long *row,
                                          unsigned long long &nb, int &ntp) {
    nb = 0ull;
    if (mk) {
        ntp = __builtin_ctzll(mk);
        mk &= mk - 1ull;
        nb = row[ntp * 32];
    }
}

template <bool B>
struct BoolTag {
    static constexpr bool value = B;
};
template <int V>
struct IntTag {
    static constexpr int value = V;
};
template <int A, int B, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (A < B) {
        f(IntTag<A>{});
        static_for<A + 1, B>(f);
    }
}

// LDS of the pair loop at KP = 16: a row of pair-table entries per point, the
// stride of 20 floats free of bank conflicts for 16-byte reads.
constexpr int PAIR_STRIDE = 20;
constexpr int PAIR_LDS_BYTES = 64 * PAIR_STRIDE * 4;
// LDS of the split operand's low parts of a wave's 64 points (padded dimension
// <= 32).
constexpr int SPLIT_LDS_BYTES = 64 * 32 * 2;
static_assert(SPLIT_LDS_BYTES <= PAIR_LDS_BYTES, "one region");

// LDS bytes of the block-wide centroid copy (padded dimension <= 128).
constexpr int CENT_LDS_BYTES = 512;

// LDS bytes of the block-wide landmark order tables (position -> landmark and
// landmark -> position, 16-bit each, two halves of equal size).
__host__ __device__ inline size_t order_lds_bytes(int g) { return (size_t)(((2 * g + 255) / 256) * 256) * 2; }

// Bytes of the screen's A operand (ntiles tiles of 32 landmarks) and of its
// LDS copy with the norms (16 per lane half and tile), 256-byte aligned.
__host__ __device__ inline size_t tile_a_bytes(int mode, int ntiles, int dc) {
    return (size_t)ntiles * dc * 64 * (mode == 1 ? 16 : 32);
}
__host__ __device__ inline size_t tile_lds_bytes(int mode, int ntiles, int dc) {
    return (tile_a_bytes(mode, ntiles, dc) + (size_t)ntiles * 128 + 255) & ~(size_t)255;
}

// Bytes of LDS one wave needs: candidate bitmaps (2 W words per lane), or for
// KP > 24 the neighbour staging of the pair loop (k entries of 10 bytes per
// lane) in the same space; then thresholds, norms and the per-lane masks of
// non-empty bitmap words.
__host__ __device__ inline int wave_smem_bytes(int kp, int k, int npair_tiles) {
    const int bits = 2 * npair_tiles * 64 * 4;
    const int nbr = kp > 24 ? k * 64 * 10 : 0;
    const int all = (bits > nbr ? bits : nbr) + 512 + 1024;
    // (kp = 16: the pair loop's rows, once the rest is done with; up to 16 the
    // split operand's low parts before the rest is written)
    const int least = kp == 16 ? PAIR_LDS_BYTES : kp < 16 ? SPLIT_LDS_BYTES : 0;
    return all < least ? least : all;
}

// Four floats at any 4-byte boundary (one 16-byte load all the same).
struct __attribute__((packed, aligned(4))) Float4U {
    float x, y, z, w;
};

// Centred values x_t - c_t of dimensions 16 c + 8 h + e (e < 8) of the point
// row xr; zero past d and for an invalid point.  Chunks of 16 dimensions within the
// row load 16 bytes at a time whatever the row's alignment.  Loaded value by value,
// the 39-dimensional rows of 842k points took the locality keys 100 us and the FP32
// fused kernel 1193; now 60 and 1059.
__device__ __forceinline__ void centred8(const float *xr, const float *centL, int d, int c, int h, bool valid,
                                         float (&v)[8]) {
    if (16 * c + 16 <= d) {
        const Float4U *x4 = reinterpret_cast<const Float4U *>(xr + 16 * c + 8 * h);
        const float4 *c4 = reinterpret_cast<const float4 *>(centL + 16 * c + 8 * h);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const Float4U q = x4[u];
            const float4 cv = c4[u];
            v[4 * u] = valid ? q.x - cv.x : 0.f;
            v[4 * u + 1] = valid ? q.y - cv.y : 0.f;
            v[4 * u + 2] = valid ? q.z - cv.z : 0.f;
            v[4 * u + 3] = valid ? q.w - cv.w : 0.f;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int d0 = 16 * c + 8 * h + e;
            v[e] = (valid && d0 < d) ? xr[d0] - centL[d0] : 0.f;
        }
    }
}

// Point index of processing slot si < n (the optional locality order).
template <int ROWS>
__device__ __forceinline__ int64_t slot_point(const EmbedArgs &a, int64_t si) {
    return ROWS == 0 && a.pt_order ? (int64_t)a.pt_order[si] : si;
}

template <int MODE, int DC>
struct PointOperand;

template <int DC>
struct PointOperand<1, DC> {  // BF16: lane holds dims 16c + 8h + e of its point
    bf16x8 b[2][DC];
};
template <int DC>
struct PointOperand<0, DC> {  // FP32: lane holds dims 16 c + 8 h + e at 8 c + e
    float b[2][8 * DC];
};

// One landmark tile's A operand and squared norms, as one lane holds them.
template <int MODE, int DC>
struct TileRegs;
template <int DC>
struct TileRegs<1, DC> {
    u32x4 a[DC];
};
template <int DC>
struct TileRegs<0, DC> {
    float a[8 * DC];
};

// The A operand and the norms come from Abase / Nbase: global memory, or the
// block's LDS copy (the caller's choice, fixed per instantiation so that the
// compiler sees the address space).
template <int MODE, int DC>
__device__ __forceinline__ void load_tile(const void *Abase, int t, int lane, TileRegs<MODE, DC> &T) {
    if constexpr (MODE == 1) {
        const u32x4 *Ap = reinterpret_cast<const u32x4 *>(Abase) + (size_t)t * DC * 64 + lane;
#pragma unroll
        for (int c = 0; c < DC; ++c) T.a[c] = Ap[c * 64];
    } else {
        const float *Ap = reinterpret_cast<const float *>(Abase) + (size_t)t * (8 * DC) * 64 + lane;
#pragma unroll
        for (int s = 0; s < 8 * DC; ++s) T.a[s] = Ap[s * 64];
    }
}

// Keys of tile t for both 32-point halves of the wave: acc[p] = |L|^2 + A B_p.
template <int MODE, int DC>
__device__ __forceinline__ void screen_tile(const float *Nbase, int t, int lane, const TileRegs<MODE, DC> &T,
                                            const PointOperand<MODE, DC> &P, f32x16 (&acc)[2]) {
    f32x16 nrm;
    {
        const float4 *np = reinterpret_cast<const float4 *>(Nbase + (size_t)(t * 2 + (lane >> 5)) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 n = np[i];
            nrm[4 * i] = n.x;
            nrm[4 * i + 1] = n.y;
            nrm[4 * i + 2] = n.z;
            nrm[4 * i + 3] = n.w;
        }
    }
    acc[0] = nrm;
    acc[1] = nrm;
    if constexpr (MODE == 1) {
#pragma unroll
        for (int c = 0; c < DC; ++c) {
            const bf16x8 av = __builtin_bit_cast(bf16x8, T.a[c]);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, P.b[0][c], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, P.b[1][c], acc[1], 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int s = 0; s < 8 * DC; ++s) {
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(T.a[s], P.b[0][s], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(T.a[s], P.b[1][s], acc[1], 0, 0, 0);
        }
    }
}

// Split BF16 keys of tile t: acc[p] = |L|^2 + Al B_p + Ah Bl_p + Ah B_p (the
// small terms first), with A = Ah + Al and B = B_p + Bl_p the high and low
// BF16 parts of the two operands.
template <int DC>
__device__ __forceinline__ void screen_tile_split(const float *Nbase, int t, int lane, const TileRegs<1, DC> &Th,
                                                  const TileRegs<1, DC> &Tl, const PointOperand<1, DC> &P,
                                                  const PointOperand<1, DC> &Pl, f32x16 (&acc)[2]) {
    f32x16 nrm;
    {
        const float4 *np = reinterpret_cast<const float4 *>(Nbase + (size_t)(t * 2 + (lane >> 5)) * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 n = np[i];
            nrm[4 * i] = n.x;
            nrm[4 * i + 1] = n.y;
            nrm[4 * i + 2] = n.z;
            nrm[4 * i + 3] = n.w;
        }
    }
    acc[0] = nrm;
    acc[1] = nrm;
#pragma unroll
    for (int c = 0; c < DC; ++c) {
        const bf16x8 al = __builtin_bit_cast(bf16x8, Tl.a[c]);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, P.b[0][c], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, P.b[1][c], acc[1], 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < DC; ++c) {
        const bf16x8 ah = __builtin_bit_cast(bf16x8, Th.a[c]);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, Pl.b[0][c], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, Pl.b[1][c], acc[1], 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < DC; ++c) {
        const bf16x8 ah = __builtin_bit_cast(bf16x8, Th.a[c]);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, P.b[0][c], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, P.b[1][c], acc[1], 0, 0, 0);
    }
}

// Cutoff weights c = 1 - exp(A (delta_q - delta_k) / delta_k) of the active
// neighbours whose FP32 value is below C_REFINE, from FP64 distances.  sk: the
// k nearest as sorted (delta^2, index) keys.  d2x(j) returns the FP64 squared
// distance from the lane's point to landmark j; it is called by all lanes
// together, with a valid landmark on every lane.  c decreases along the sorted
// list, so the weights to refine are the lane's last nref active ones: on
// return cref[r-1] holds the weight of neighbour kact - r for r = 1..nref
// (nref <= N_REFINE).  Returns R_NEARTIE when the FP64 distances order a
// refined neighbour after the k-th (the exact path then ranks the point again)
// and R_ILLCOND when more than N_REFINE weights need it (rare: 0.03% of the
// points of 1M x 32-D with 400 landmarks even at k = 16).
template <int KP, class D2X>
__device__ __forceinline__ unsigned refine_cutoffs(const EmbedArgs &a, const double (&sk)[KP], bool valid,
                                                   D2X &&d2x, float (&cref)[N_REFINE], int &nref) {
    nref = 0;
#pragma unroll
    for (int r = 0; r < N_REFINE; ++r) cref[r] = 0.f;
    if (!a.use_cutoff) return 0u;
    float d2k = 0.f;
    int jk = 0;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        if (q == a.k - 1) {
            d2k = key_d2(sk[q]);
            jk = key_idx(sk[q]);
        }
    }
    // c < C_REFINE  <=>  delta_q / delta_k > 1 + ln(1 - C_REFINE) / A
    const float f = 1.f + LN_1M_CREFINE / a.cutoff;
    const float lim = f > 0.f ? d2k * f * f : 0.f;
#pragma unroll
    for (int q = 0; q < KP; ++q)
        if (valid && q < a.kact && key_d2(sk[q]) > lim) ++nref;
    unsigned reason = 0u;
    if (nref > N_REFINE) {
        reason |= R_ILLCOND;
        nref = N_REFINE;
    }
    if (__ballot(nref > 0) == 0ull) return reason;
    const double d2k64 = d2x(jk);
    const float dk32 = __builtin_amdgcn_sqrtf((float)d2k64);
#pragma unroll
    for (int r = 1; r <= N_REFINE; ++r) {
        if (__ballot(r <= nref) == 0ull) break;
        const bool act = r <= nref;
        int jt = jk;
#pragma unroll
        for (int q = 0; q < KP; ++q)
            if (act && q == a.kact - r) jt = key_idx(sk[q]);
        const double d2t = d2x(jt);
        // only the difference needs FP64: it keeps its relative accuracy
        // through the conversion, and the rest is well conditioned
        const float dd = (float)(d2t - d2k64);
        const float den = (__builtin_amdgcn_sqrtf((float)d2t) + dk32) * dk32;
        const float z = den > 0.f ? a.cutoff * dd / den : 0.f;
        if (act && (d2t > d2k64 || (d2t == d2k64 && jt > jk))) reason |= R_NEARTIE;
        cref[r - 1] = one_minus_exp(z);
    }
    return reason;
}

// Phase C for one point (lane): scores from the k sorted distances, the pair
// terms, the FP64 2x2 solve and the output store.  sk holds the k nearest as
// packed (delta^2, index) keys, ascending.  Returns the accumulated fallback
// reasons; the output is written only when there is none.
// The cutoff weight of neighbour kact - r comes from cref[r-1] for r = 1..nref
// (see refine_cutoffs).
template <int KP>
__device__ __forceinline__ unsigned project_point(const EmbedArgs &a, const double (&sk)[KP],
                                                  int lane, bool valid, long long pi, unsigned reason,
                                                  float *nbD2, float *nbS, unsigned short *nbI,
                                                  const unsigned short *iposL, const float (&cref)[N_REFINE],
                                                  int nref) {
    float d2q[KP], dl[KP], sq[KP], lxq[KP], lyq[KP];
    int jq[KP];
    float mu = 0.f;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        d2q[q] = (q < a.k) ? key_d2(sk[q]) : 0.f;
        jq[q] = (q < a.k) ? key_idx(sk[q]) : 0;
        dl[q] = __builtin_amdgcn_sqrtf(d2q[q]);
        if (q < a.k) mu = fmaf(dl[q], 1.f / (float)(q + 1), mu);
    }
    float d2k = d2q[0];
#pragma unroll
    for (int q = 0; q < KP; ++q)
        if (q == a.k - 1) d2k = d2q[q];
    mu /= a.Wk;
    float var = 0.f;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        if (q < a.k) {
            const float e = dl[q] - mu;
            var = fmaf(e * e, 1.f / (float)(q + 1), var);
        }
    }
    var /= a.Wk;
    const float dk = __builtin_amdgcn_sqrtf(d2k);
    // cutoff argument A (delta_q - delta_k) / delta_k from the FP32 distances
    const float cut_scale = a.cutoff * __builtin_amdgcn_rcpf(dk);
    const bool degenerate = d2q[0] == d2k;
    const bool flat = !(var > 1e-30f * mu * mu);
    const float isig = flat ? 0.f : a.boost * rsqrtf(var);
    if (degenerate) reason |= R_DEGEN;
    const float ox = a.l2d[2 * jq[0]], oy = a.l2d[2 * jq[0] + 1];
    float ssum = 0.f;
    float M00 = 0.f, M01 = 0.f, M11 = 0.f, r0 = 0.f, r1 = 0.f;
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        const float2 lv = reinterpret_cast<const float2 *>(a.l2d)[jq[q]];
        lxq[q] = lv.x - ox;
        lyq[q] = lv.y - oy;
    }
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        sq[q] = 0.f;
        if (q < a.k) {
            const float e = flat ? 1.f : __expf((mu - dl[q]) * isig);
            float c = a.use_cutoff ? 1.f - __expf((dl[q] - dk) * cut_scale) : 1.f;
            if constexpr (KP <= 8) {
#pragma unroll
                for (int r = 1; r <= N_REFINE; ++r)
                    if (r <= nref && q == a.kact - r) c = cref[r - 1];
            }
            sq[q] = degenerate ? 0.f : e * c;
            ssum += sq[q];
            const float gs = a.gravity * sq[q];
            M00 += gs;
            M11 += gs;
            r0 = fmaf(gs, lxq[q], r0);
            r1 = fmaf(gs, lyq[q], r1);
        }
    }
    if (!(ssum > 0.f)) reason |= R_DEGEN;

    // pairs (i < j among the neighbours with non-zero score); d2i <= d2j.  The
    // pair (i, j) adds q/|h|^2 h h^T to M and q/|h|^2 h t to r, with h = l_j - l_i,
    // t = D |h|^2 + h.l_i and D its segment coordinate.  Split as q D h plus
    // (q/|h|^2 h h^T) l_i, the second part sums over j into M_i l_i, so a pair
    // costs no dot product; s_i multiplies the sums of base i once.  The pair
    // table supplies 1/(2|L_u - L_v|^2), 0 for coincident landmarks; 1/|h|^2
    // comes from the 2-D difference at hand, and a pair with either length 0
    // gets weight 0, so a skipped pair adds exactly 0.
    float pmax = 0.f;  // largest delta_j^2 / (2 |L_i - L_j|^2) over the pairs
    const bool unit_adjust = a.adjust == 1.0f;
    auto pair_term = [&](auto unit, float d2i, float lxi, float lyi, float d2j, float sj, float lxj,
                         float lyj, float inv, float (&Mi)[3], float (&ri)[2]) {
        const float hx = lxj - lxi, hy = lyj - lyi;
        const float hh = fmaf(hx, hx, hy * hy);
        const float ihh = (inv > 0.f && hh > 0.f) ? __builtin_amdgcn_rcpf(hh) : 0.f;
        const float D = fmaf(d2i - d2j, inv, 0.5f);
        pmax = fmaxf(pmax, d2j * inv);
        // n = h / |h|^2: M += s_j n n^T, r += s_j D n (times |h|^(2 - 2 adjust))
        const float nx = hx * ihh, ny = hy * ihh;
        float tx, ty;
        // unit: adjust == 1 (weight 1 / |h|^2), as a compile-time tag so that
        // the two variants of the pair loop are separate code
        if constexpr (decltype(unit)::value) {
            tx = sj * nx;
            ty = sj * ny;
        } else {
            const float q = ihh > 0.f ? sj * exp2f(a.adjust * __log2f(ihh)) : 0.f;
            tx = q * hx;
            ty = q * hy;
        }
        Mi[0] = fmaf(tx, nx, Mi[0]);
        Mi[1] = fmaf(tx, ny, Mi[1]);
        Mi[2] = fmaf(ty, ny, Mi[2]);
        ri[0] = fmaf(tx, D, ri[0]);
        ri[1] = fmaf(ty, D, ri[1]);
    };
    // closes base i: r += s_i (r_i + M_i l_i), M += s_i M_i
    auto close_base = [&](bool origin, float si, float lxi, float lyi, const float (&Mi)[3],
                          float (&ri)[2]) {
        if (!origin) {
            ri[0] = fmaf(Mi[0], lxi, fmaf(Mi[1], lyi, ri[0]));
            ri[1] = fmaf(Mi[1], lxi, fmaf(Mi[2], lyi, ri[1]));
        }
        M00 = fmaf(si, Mi[0], M00);
        M01 = fmaf(si, Mi[1], M01);
        M11 = fmaf(si, Mi[2], M11);
        r0 = fmaf(si, ri[0], r0);
        r1 = fmaf(si, ri[1], r1);
    };
    auto run_pairs = [&](auto unit) {
    if constexpr (KP == 16) {
        // The pair-table reads by 16 lanes a point, four points a load.  Step t
        // reads the rows of bases t and 14 - t, which have 16 entries together:
        // lane v > t the entry (t, v), lane v <= t the entry (14 - t, 15 - v).  The
        // neighbours sit close together in the landmark order, so a point's
        // entries of a row fall into two or three lines, which this asks for once;
        // a lane that read its own point's entries one by one asked for them
        // 15 - u times, mostly while they were still on their way.  The entries
        // go through LDS to their points' lanes, one step ahead of use.  At 1M x
        // 32-D the L1's line accesses fell from 159M to 136M a call; the address
        // arithmetic takes back most of it there (0.5 to 1% faster), projections
        // from cached neighbours are 4% faster.
        const char *ptab = reinterpret_cast<const char *>(a.pairs);
        float *rows = nbD2;  // 64 x PAIR_STRIDE
        const int v16 = lane & 15;
        unsigned col[16];    // 4 x position of neighbour v16 of point 4 G + (lane / 16)
        {
            unsigned *pk = reinterpret_cast<unsigned *>(rows);  // 64 x 16 positions of 16 bits
            const unsigned p0 = iposL[jq[0]];
#pragma unroll
            for (int q = 0; q < 16; q += 2) {
                // slots past the active neighbours repeat the first
                const unsigned lo = q < a.kact ? iposL[jq[q]] : p0, hi = q + 1 < a.kact ? iposL[jq[q + 1]] : p0;
                pk[lane * 8 + q / 2] = lo | (hi << 16);
            }
            wave_lds_fence();
            const unsigned short *ps = reinterpret_cast<const unsigned short *>(rows) + lane;
#pragma unroll
            for (int G = 0; G < 16; ++G) col[G] = 4u * ps[64 * G];
            wave_lds_fence();
        }
        float ld[16];
        auto fetch = [&](auto tt) {
            constexpr int T = decltype(tt)::value;
            const bool up = v16 > T;
#pragma unroll
            for (int G = 0; G < 16; ++G) {
                const unsigned rt = row16_bcast<T>(col[G]), rm = row16_bcast<14 - T>(col[G]);
                const unsigned cm = (unsigned)__builtin_amdgcn_mov_dpp((int)col[G], 0x140, 0xf, 0xf, true);  // lane 15 - v
                ld[G] = *reinterpret_cast<const float *>(
                    ptab + (size_t)(__umul24(up ? rt : rm, (unsigned)a.g) + (up ? col[G] : cm)));
            }
        };
        fetch(IntTag<0>{});
        float *wr = rows + (lane >> 4) * PAIR_STRIDE + v16;
        const float4 *rd = reinterpret_cast<const float4 *>(rows + lane * PAIR_STRIDE);
        static_for<0, 8>([&](auto tt) {
            constexpr int T = decltype(tt)::value;
#pragma unroll
            for (int G = 0; G < 16; ++G) wr[4 * G * PAIR_STRIDE] = ld[G];
            wave_lds_fence();
            if constexpr (T + 1 < 8) fetch(IntTag<T + 1>{});
            float pv[16];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 v = rd[i];
                pv[4 * i] = v.x;
                pv[4 * i + 1] = v.y;
                pv[4 * i + 2] = v.z;
                pv[4 * i + 3] = v.w;
            }
            wave_lds_fence();
            auto base = [&](auto ut) {
                constexpr int U = decltype(ut)::value;
                if (U < a.kact - 1) {
                    float Mi[3] = {0.f, 0.f, 0.f}, ri[2] = {0.f, 0.f};
#pragma unroll
                    for (int qj = U + 1; qj < 16; ++qj)
                        if (qj < a.kact)
                            pair_term(unit, d2q[U], lxq[U], lyq[U], d2q[qj], sq[qj], lxq[qj], lyq[qj],
                                      pv[U == T ? qj : 15 - qj], Mi, ri);
                    // neighbour 0 is the origin of the 2-D frame
                    close_base(U == 0, sq[U], lxq[U], lyq[U], Mi, ri);
                }
            };
            base(tt);
            if constexpr (T < 7) base(IntTag<14 - T>{});
        });
    } else if constexpr (KP <= 24) {
        // neighbour data in registers (fully unrolled: 276 pair slots at
        // k <= 24, which ran 6% faster at 1M x 48-D, 1024 landmarks, k = 20
        // than the LDS staging below); each row of pair-table loads is issued
        // together, unconditionally (slots past k hold landmark 0, a valid
        // entry, and are never used), addressed by 32-bit byte offsets from
        // the table base (g <= 4096: under 2^26 bytes)
        const char *ptab = reinterpret_cast<const char *>(a.pairs);
#pragma unroll
        for (int qi = 0; qi < KP - 1; ++qi) {
            if (qi < a.kact - 1) {
                const unsigned rowoff = mul24(iposL[jq[qi]], (unsigned)a.g);
                float pv[KP];
#pragma unroll
                for (int qj = qi + 1; qj < KP; ++qj)
                    pv[qj] = *reinterpret_cast<const float *>(ptab + (size_t)((rowoff + iposL[jq[qj]]) * 4u));
                float Mi[3] = {0.f, 0.f, 0.f}, ri[2] = {0.f, 0.f};
#pragma unroll
                for (int qj = qi + 1; qj < KP; ++qj)
                    if (qj < a.kact)
                        pair_term(unit, d2q[qi], lxq[qi], lyq[qi], d2q[qj], sq[qj], lxq[qj], lyq[qj],
                                  pv[qj], Mi, ri);
                // neighbour 0 is the origin of the 2-D frame
                close_base(qi == 0, sq[qi], lxq[qi], lyq[qi], Mi, ri);
            }
        }
    } else {
        // larger neighbourhoods: neighbour data through LDS, inner loop unrolled
        // by 4.  The table is symmetric; entry (u, v) is read at row min(u, v),
        // column max(u, v), so a point's reads cover fewer cache lines (each
        // row only to the right of its own position): 4% faster at 1M x 48-D,
        // 1024 landmarks, k = 20 when this path served that shape.  (With
        // k <= 16 the extra address arithmetic cost more than it saved.)
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            if (q < a.k) {
                nbD2[q * 64 + lane] = d2q[q];
                nbS[q * 64 + lane] = sq[q];
                nbI[q * 64 + lane] = (unsigned short)jq[q];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (int qi = 0; qi < a.kact - 1; ++qi) {
            const float d2i = nbD2[qi * 64 + lane], si = nbS[qi * 64 + lane];
            const int ui = nbI[qi * 64 + lane];
            const float2 li = reinterpret_cast<const float2 *>(a.l2d)[ui];
            const float lxi = li.x - ox, lyi = li.y - oy;
            const unsigned pu = iposL[ui];
            float Mi[3] = {0.f, 0.f, 0.f}, ri[2] = {0.f, 0.f};
            for (int qb = qi + 1; qb < a.kact; qb += 4) {
                float pv[4];
                float d2j[4], sj[4], lxj[4], lyj[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int qj = qb + u;
                    const bool ok = qj < a.kact;
                    const int vj = ok ? nbI[qj * 64 + lane] : 0;
                    const unsigned pw = iposL[vj];
                    pv[u] = ok ? a.pairs[(size_t)min(pu, pw) * a.g + max(pu, pw)] : 0.f;
                    d2j[u] = ok ? nbD2[qj * 64 + lane] : 0.f;
                    sj[u] = ok ? nbS[qj * 64 + lane] : 0.f;
                    const float2 lv = reinterpret_cast<const float2 *>(a.l2d)[vj];
                    lxj[u] = lv.x - ox;
                    lyj[u] = lv.y - oy;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    pair_term(unit, d2i, lxi, lyi, d2j[u], sj[u], lxj[u], lyj[u], pv[u], Mi, ri);
            }
            close_base(false, si, lxi, lyi, Mi, ri);
        }
        __builtin_amdgcn_wave_barrier();
    }
    };
    if (unit_adjust)
        run_pairs(BoolTag<true>{});
    else
        run_pairs(BoolTag<false>{});
    const bool ill = pmax > ILL_PAIR;
    // 2x2 solve in FP64 (Cramer's rule)
    const double m00 = M00, m01 = M01, m11 = M11, rr0 = r0, rr1 = r1;
    const double det = m00 * m11 - m01 * m01;
    const double tr = m00 + m11;
    if (ill || !(det > 0.0) || 0.25 * tr * tr > ILL_COND * det) reason |= R_ILLCOND;
    if (valid && reason == 0) {
        const double px = (rr0 * m11 - m01 * rr1) / det;
        const double py = (m00 * rr1 - m01 * rr0) / det;
        reinterpret_cast<float2 *>(a.out)[pi] = make_float2((float)((double)ox + px),
                                                            (float)((double)oy + py));
    }
    return reason;
}

// Lists a point for the exact path, from the front, or (order alone open) for
// embed_reorder, from the back.
__device__ __forceinline__ void list_point(const EmbedArgs &a, int64_t pi, unsigned reason, float thr) {
    if (reason == R_ORDER && a.order_list) {
        const int64_t slot = a.fb_cap - 1 - (int64_t)atomicAdd(&a.counters[C_ORD_LEN], 1ull);
        a.fb_list[slot] = (int32_t)pi;
        a.fb_reason[slot] = (uint8_t)R_NEARTIE;
        return;
    }
    if (reason & R_ORDER) reason = (reason & ~(unsigned)R_ORDER) | R_NEARTIE;
    const unsigned long long slot = atomicAdd(&a.counters[C_FB_LEN], 1ull);
    a.fb_list[slot] = (int32_t)pi;
    a.fb_reason[slot] = (uint8_t)reason;
    a.fb_thresh[slot] = thr;
}

// Projection only (phases of scores, pairs and solve) from given k nearest
// landmarks (knn_idx / knn_d2, sorted by (distance, index)), e.g. cached from
// an earlier call with the same high-dimensional landmarks.
template <int KP>
__global__ void __launch_bounds__(256) embed_project(EmbedArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wpb = blockDim.x >> 6;
    unsigned char *wsm = smem + (size_t)wave * (KP * 64 * 10);
    float *nbD2 = reinterpret_cast<float *>(wsm);
    float *nbS = nbD2 + KP * 64;
    unsigned short *nbI = reinterpret_cast<unsigned short *>(nbS + KP * 64);
    unsigned short *iposL = reinterpret_cast<unsigned short *>(smem + (size_t)wpb * (KP * 64 * 10));
    for (int e = threadIdx.x; e < a.g; e += blockDim.x) iposL[e] = (unsigned short)a.ipos[e];
    __syncthreads();
    const int64_t nwt = (a.n + 63) / 64;
    // Tile wt goes to block wt mod grid, wave (wt / grid) mod wpb: the last,
    // partial round of tiles then spreads over all blocks (CUs) instead of
    // filling the first few.
    for (int64_t wt = (int64_t)wave * gridDim.x + blockIdx.x; wt < nwt; wt += (int64_t)gridDim.x * wpb) {
        const int64_t pi = wt * 64 + lane;
        const bool valid = pi < a.n;
        // A cached index outside [0, g) (the exact path writes -1 for a point
        // without k finite distances) is never used for a load: it becomes
        // landmark 0 and the point goes to the exact path, which ranks it again.
        double sk[KP];
        bool bad_idx = false;
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            sk[q] = INFINITY;
            if (valid && q < a.k) {
                int j = a.knn_idx[pi * a.k + q];
                if (j < 0 || j >= a.g) {
                    bad_idx = true;
                    j = 0;
                }
                sk[q] = pack_key(a.knn_d2[pi * a.k + q], j);
            }
        }
        const unsigned mark = valid && a.knn_mark ? a.knn_mark[pi] : 0u;
        unsigned reason = mark == 0u ? 0u : mark == 2u ? (unsigned)R_ORDER : (unsigned)R_NEARTIE;
        if (bad_idx) reason |= R_UNCERT;
        float d2k = INFINITY;
#pragma unroll
        for (int q = 0; q < KP; ++q)
            if (q == a.k - 1) d2k = key_d2(sk[q]);
        const float thr = kth_bound(d2k, a.dp);
        const float *xr = a.X + (valid ? pi : 0) * a.ldx;
        auto d2x = [&](int jl) -> double {
            const float *Lr = a.Lpad + (size_t)iposL[jl] * a.dp;
            double sum[4] = {0.0, 0.0, 0.0, 0.0};  // as the fused kernel sums
            for (int t0 = 0; t0 < a.d; t0 += 16)
#pragma unroll
                for (int t = 0; t < 16; ++t) {
                    const double e = t0 + t < a.d ? (double)xr[t0 + t] - (double)Lr[t0 + t] : 0.0;
                    sum[t / 4] = fma(e, e, sum[t / 4]);
                }
            return (sum[0] + sum[1]) + (sum[2] + sum[3]);
        };
        float cref[N_REFINE] = {};
        int nref = 0;
        if constexpr (KP <= 8) reason |= refine_cutoffs<KP>(a, sk, valid, d2x, cref, nref);
        reason = project_point<KP>(a, sk, lane, valid, pi, reason, nbD2, nbS, nbI, iposL, cref, nref);
        if (valid && reason) list_point(a, pi, reason, thr);
    }
}

// ROWS = 1: the block stages the padded landmark rows in LDS for the exact
// rescoring (a.lds_rows); ROWS = 0: rows stream from memory.  The two are
// separate instantiations so that each gets its own register allocation.
// KF = 1: k == KP and k < g (so k - 1 neighbours are active), known at
// compile time: the loops over the sorted list and the pairs lose their
// bounds tests (5% faster at 1M x 32-D with k = 16, 4% at 10M x 64-D).
// KP = 1 (KF = 1 only): the nearest landmark of the landmark update, with no
// projection.  1M x 32-D, 400 landmarks: 460 us with the 8-entry list of the k <=
// 8 kernel in FP32 mode, now 150 us.
template <int MODE, int DC, int KP, int ROWS, int KF>
__global__ void __launch_bounds__(main_max_block(MODE, DC, KP)) embed_main(EmbedArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    if constexpr (KF == 1) {
        a.k = KP;
        a.kact = KP - 1;
    }
    constexpr int DP = 16 * DC;
    constexpr int RS = DP + 4;  // LDS row stride (floats): spreads rows over the banks
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wpb = blockDim.x >> 6;
    const int h = lane >> 5;
    const int i32 = lane & 31;
    const int W = a.npair_tiles;
    // Block-wide copies: the centroid (read for every point group), and
    // optionally the landmark rows for exact rescoring.
    float *centL = reinterpret_cast<float *>(smem);
    const size_t tab_bytes = order_lds_bytes(a.g);
    unsigned short *permL = reinterpret_cast<unsigned short *>(smem + CENT_LDS_BYTES);
    unsigned short *iposL = permL + tab_bytes / 4;
    float *rowsL = reinterpret_cast<float *>(smem + CENT_LDS_BYTES + tab_bytes);
    const size_t rows_bytes = ROWS ? (((size_t)a.g * RS * 4 + 255) & ~(size_t)255) : 0;
    // optionally the screen operands (A tiles and norms), read by every wave
    // twice per 64 points
    const size_t a_bytes = tile_a_bytes(MODE, a.ntiles, DC);
    const size_t tiles_bytes = a.lds_tiles ? tile_lds_bytes(MODE, a.ntiles, DC) : 0;
    unsigned char *tilesL = smem + CENT_LDS_BYTES + tab_bytes + rows_bytes;
    const float *normsL = reinterpret_cast<const float *>(tilesL + a_bytes);
    for (int e = threadIdx.x; e < DP; e += blockDim.x) centL[e] = e < a.d ? a.cent[e] : 0.f;
    for (int e = threadIdx.x; e < a.g; e += blockDim.x) {
        permL[e] = (unsigned short)a.perm[e];
        iposL[e] = (unsigned short)a.ipos[e];
    }
    if constexpr (ROWS == 1) {
        for (int e = threadIdx.x; e < a.g * (DP / 4); e += blockDim.x) {
            const int j = e / (DP / 4), q = e % (DP / 4);
            reinterpret_cast<float4 *>(rowsL + (size_t)j * RS)[q] =
                reinterpret_cast<const float4 *>(a.Lpad + (size_t)j * DP)[q];
        }
    }
    if (a.lds_tiles) {
        const size_t nv = (a_bytes + (size_t)a.ntiles * 128) / 16;
        const float4 *srcA = reinterpret_cast<const float4 *>(a.A);
        const float4 *srcN = reinterpret_cast<const float4 *>(a.norms);
        for (size_t e = threadIdx.x; e < nv; e += blockDim.x)
            reinterpret_cast<float4 *>(tilesL)[e] = e < a_bytes / 16 ? srcA[e] : srcN[e - a_bytes / 16];
    }
    __syncthreads();
    unsigned char *wsm = smem + CENT_LDS_BYTES + tab_bytes + rows_bytes + tiles_bytes +
                         (size_t)wave * wave_smem_bytes(KP, a.k, W);
    unsigned *bitsL = reinterpret_cast<unsigned *>(wsm);
    float *nbD2 = reinterpret_cast<float *>(wsm);
    float *nbS = nbD2 + a.k * 64;
    unsigned short *nbI = reinterpret_cast<unsigned short *>(nbS + a.k * 64);
    const int nbr_bytes = KP > 24 ? a.k * 64 * 10 : 0;
    const int tail = (2 * W * 64 * 4 > nbr_bytes) ? 2 * W * 64 * 4 : nbr_bytes;
    float *certL = reinterpret_cast<float *>(wsm + tail);  // 64 certificate bounds (512 B reserved)
    unsigned long long *maskL = reinterpret_cast<unsigned long long *>(certL + 128);

    // points in locality order (launched with ROWS = 0 and no LDS tiles)
    const bool ordered = ROWS == 0 && a.pt_order;
    const float lmax = a.lmax[0];
    const float qa = a.lmax[1];  // max_j |bf16(-2 (L_j - c)) + 2 (L_j - c)|

    unsigned long long st_cand = 0;
    const int64_t nwt = (a.n + 63) / 64;
    // Tile wt goes to block wt mod grid, turn (wt / grid) mod wpb: the last,
    // partial round of tiles then spreads over all blocks (CUs) instead of
    // filling the first few.  Each block on a CU starts one SIMD after the one
    // before it (seen in the times of such launches), so in blocks of 4 waves the
    // turns go to the waves such that a CU's m-th tile runs on SIMD m mod 4.  70k
    // points x 128-D, 400 landmarks, k = 16, two blocks a CU: 194 us a call with turn
    // = wave in full blocks, 172 so.
    int turn = wave;
    if (wpb == 4) {
        const int layers = (int)((gridDim.x + (unsigned)a.cus - 1u) / (unsigned)a.cus);
        const int common = layers & 1 ? 1 : layers & 2 ? 2 : 4;  // of layers and 4
        for (int u = 0; u < 4; ++u)
            if (((u * layers + u * common / 4) & 3) == wave) turn = u;
    }
    for (int64_t wt = (int64_t)turn * gridDim.x + blockIdx.x; wt < nwt; wt += (int64_t)gridDim.x * wpb) {
        const int64_t pbase = wt * 64;

        // ---------------- point operands (centred), and |x - c|^2.  Pass 1
        // always runs on the BF16 operand; FP32 mode builds its FP32 operand
        // for pass 2 afterwards.
        PointOperand<1, DC> P16, P16lo;  // P16lo: BF16 mode's pass 2
        float xnp[2], dxp[2];  // |x - c|^2 and |bf16(x - c) - (x - c)|^2
        float nlo[2], nre[2];  // BF16 mode: |lo| and |r| of the split (see e2)
        // Low parts of two split values from their remainders after the high
        // parts, adding to |lo|^2 and |r|^2.  BF16 mode forms them with the high
        // parts and holds them through pass 1 in registers, or where 12 waves
        // leave none in the wave's LDS, which pass 2 writes afterwards (not with
        // points in locality order, whose pass 1 uses it, nor beyond 64 padded
        // dimensions: there the rows are read again; at 1M x 32-D that took 11K of
        // the tile's 112K cycles).
        constexpr bool SPLIT_STASH = MODE == 1 && main_max_block(MODE, DC, KP) == 768 && ROWS == 1;
        constexpr bool SPLIT_EARLY = SPLIT_STASH || (MODE == 1 && main_max_block(MODE, DC, KP) == 512 && DC <= 4);
        u32x4 *stash = reinterpret_cast<u32x4 *>(wsm) + lane;
        auto split_low = [](float r0, float r1, float &lsum, float &rsum) -> unsigned {
            const unsigned lw = bf16_pair(r0, r1);
            const float l0 = bf16_lo(lw), l1 = bf16_hi(lw);
            lsum = fmaf(l0, l0, lsum);
            lsum = fmaf(l1, l1, lsum);
            rsum = fmaf(r0 - l0, r0 - l0, rsum);
            rsum = fmaf(r1 - l1, r1 - l1, rsum);
            return lw;
        };
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int64_t si = pbase + 32 * p + i32;
            const bool valid = si < a.n;
            const float *xr = a.X + (valid ? slot_point<ROWS>(a, si) : 0) * a.ldx;
            float part = 0.f, dpart = 0.f, lpart = 0.f, rpart = 0.f;
#pragma unroll
            for (int c = 0; c < DC; ++c) {
                float v[8];
                centred8(xr, centL, a.d, c, h, valid, v);
                unsigned w[4], lw[4];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    part = fmaf(v[e], v[e], part);
                    part = fmaf(v[e + 1], v[e + 1], part);
                    const unsigned hw = bf16_pair(v[e], v[e + 1]);
                    // quantisation errors (exact in FP32)
                    const float q0 = v[e] - bf16_lo(hw), q1 = v[e + 1] - bf16_hi(hw);
                    dpart = fmaf(q0, q0, dpart);
                    dpart = fmaf(q1, q1, dpart);
                    w[e >> 1] = hw;
                    if constexpr (SPLIT_EARLY) lw[e >> 1] = split_low(q0, q1, lpart, rpart);
                }
                P16.b[p][c] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
                if constexpr (SPLIT_STASH)
                    stash[(p * DC + c) * 64] = u32x4{lw[0], lw[1], lw[2], lw[3]};
                else if constexpr (SPLIT_EARLY)
                    P16lo.b[p][c] = __builtin_bit_cast(bf16x8, u32x4{lw[0], lw[1], lw[2], lw[3]});
            }
            xnp[p] = part + __shfl_xor(part, 32);
            dxp[p] = dpart + __shfl_xor(dpart, 32);
            if constexpr (SPLIT_EARLY) {
                nlo[p] = sqrtf(lpart + __shfl_xor(lpart, 32));
                nre[p] = sqrtf(rpart + __shfl_xor(rpart, 32));
            }
        }
        // Rigorous bounds of the screen's rounding error in key units, per
        // point.  With a = -2(L - c) and its BF16 image a + da, x' = x - c and
        // its BF16 image x' + dx: |x'.da + dx.a + dx.da| <= |x'| max|da| + |dx|
        // (max|a| + max|da|) (|dx| exact per point, max|da| from the
        // preparation); plus FP32 accumulation and centring, (2 d_pad + 16) u
        // (|x'| + max|L - c|)^2.  FP32 operands are exact and 2 (2u + u^2) |x'|
        // max|L - c| bounds their products.  The FP32 evaluation of the bound
        // is covered by the factor 1.01.  (The split BF16 keys of pass 2 have
        // their own bound, e2 below.)
        float e16[2], e32[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const float sx = sqrtf(xnp[p]);
            const float facc = (2.f * DP + 16.f) * U32 * (sx + lmax) * (sx + lmax);
            e16[p] = 1.01f * (sx * qa + sqrtf(dxp[p]) * (2.f * lmax + qa) + facc);
            e32[p] = 1.01f * (2.f * (2.f * U32 + U32 * U32) * sx * lmax + facc);
        }

        // ---------------- pass 1: group minima of the BF16 keys; |x - c|^2 is
        // added once per group afterwards (rounding is monotone, so the
        // minimum of the sums equals the sum with the minimum).
        float gmin[2][2][16];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int r = 0; r < 16; ++r) gmin[p][q][r] = INFINITY;
        const float ninf = opaque_neg_inf();
        auto pass1_consume = [&](const f32x16 (&acc)[2], int half) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int r = 0; r < 16; ++r) gmin[p][half][r] = vmin32(gmin[p][half][r], acc[p][r], ninf);
        };
        // one screen pass over all tiles with the operand of precision OM,
        // tiles from the block's LDS copy or from global memory
        auto screen_pass = [&](auto in_lds, auto opm, const auto &Pop, const void *Aglob, auto consume,
                               auto store) {
            constexpr int OM = decltype(opm)::value;
            const void *Ab = decltype(in_lds)::value ? static_cast<const void *>(tilesL) : Aglob;
            const float *Nb = decltype(in_lds)::value ? normsL : a.norms;
            TileRegs<OM, DC> T;
            for (int tp = 0; tp < W; ++tp) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    f32x16 acc[2];
                    load_tile<OM, DC>(Ab, 2 * tp + half, lane, T);
                    screen_tile<OM, DC>(Nb, 2 * tp + half, lane, T, Pop, acc);
                    consume(acc, half);
                }
                store(tp);
            }
        };
        // BF16 mode's pass 2: split operands, high parts from LDS or global
        // memory, low parts from global memory (a.A16)
        auto screen_pass_split = [&](auto in_lds, auto consume, auto store) {
            const void *Ab = decltype(in_lds)::value ? static_cast<const void *>(tilesL) : a.A;
            const float *Nb = decltype(in_lds)::value ? normsL : a.norms;
            // the low parts one tile ahead (their latency took 8K cycles a wave at
            // 1M x 32-D, where the high parts are in LDS)
            TileRegs<1, DC> Th, Tl[2];
            // (beyond 64 dimensions it takes registers from the operands: 200k x 128-D,
            // 400 landmarks, k = 16, 353 us ahead, 344 not)
            constexpr bool AHEAD = DC <= 4;
            if constexpr (AHEAD) load_tile<1, DC>(a.A16, 0, lane, Tl[0]);
            for (int tp = 0; tp < W; ++tp) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int t = 2 * tp + half;
                    f32x16 acc[2];
                    if constexpr (AHEAD)
                        load_tile<1, DC>(a.A16, t + 1 < 2 * W ? t + 1 : t, lane, Tl[1 - half]);
                    else
                        load_tile<1, DC>(a.A16, t, lane, Tl[half]);
                    load_tile<1, DC>(Ab, t, lane, Th);
                    screen_tile_split<DC>(Nb, t, lane, Th, Tl[half], P16, P16lo, acc);
                    consume(acc, half);
                }
                store(tp);
            }
        };
        // Points in locality order: a wavefront's points share a neighbourhood,
        // and most tiles hold no candidate of theirs.  Pass 1 then also keeps,
        // per lane and tile, the smallest approximate delta^2 (key + |x - c|^2)
        // of both points, rounded down to 16 bits, in the words where pass 2 will
        // put the tile's candidate bits: the word of (p = half, tp) holds tile
        // 2 tp + half's two values.  A pass-1 key is within E16 of the exact key,
        // so a 32-point half whose values all exceed its points' tau + E16 + E2
        // (pass-2 keys then exceed tau) has no candidate in that tile, and pass 2
        // leaves the tile out for it.
        auto tile_word = [&](int half, int tp) -> unsigned & { return bitsL[((half * W + tp) * 32 + i32) * 2 + h]; };
        auto screen_pass1_tiles = [&](const void *Ab) {
            const float *Nb = a.norms;
            TileRegs<1, DC> T;
            for (int tp = 0; tp < W; ++tp) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    f32x16 acc[2];
                    load_tile<1, DC>(Ab, 2 * tp + half, lane, T);
                    screen_tile<1, DC>(Nb, 2 * tp + half, lane, T, P16, acc);
                    pass1_consume(acc, half);
                    unsigned v[2];
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        float m = acc[p][0];
#pragma unroll
                        for (int r = 1; r < 16; ++r) m = vmin32(m, acc[p][r], ninf);
                        v[p] = (unsigned)max(__float_as_int(m + xnp[p]), 0);
                    }
                    tile_word(half, tp) = (v[0] >> 16) | (v[1] & 0xFFFF0000u);
                }
            }
        };
        // pass 2 over the tiles that may hold candidates; thr16: tau + E16 + E2
        // as an approximate delta^2, its upper 16 bits (rounding is monotone, so
        // a larger stored value means a larger key)
        auto screen_pass2_tiles = [&](const auto &P32, auto consume, auto store, const unsigned (&thr16)[2]) {
            const void *Ab = a.A;
            const float *Nb = a.norms;
            for (int tp = 0; tp < W; ++tp) {
                bool need[2][2];
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const unsigned v = tile_word(half, tp);
                    need[half][0] = __ballot((v & 0xFFFFu) <= thr16[0]) != 0ull;
                    need[half][1] = __ballot((v >> 16) <= thr16[1]) != 0ull;
                }
                if (!(need[0][0] || need[0][1] || need[1][0] || need[1][1])) continue;  // the masks leave these words out
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int t = 2 * tp + half;
                    f32x16 acc[2];
                    if (need[half][0] || need[half][1]) {
                        const float4 *np = reinterpret_cast<const float4 *>(Nb + (size_t)(t * 2 + (lane >> 5)) * 16);
                        float4 n[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) n[i] = np[i];
                        TileRegs<MODE, DC> T;
                        TileRegs<1, DC> Tl;  // BF16 mode: the low parts
                        load_tile<MODE, DC>(Ab, t, lane, T);
                        if constexpr (MODE == 1) load_tile<1, DC>(a.A16, t, lane, Tl);
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            if (!need[half][p]) continue;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                acc[p][4 * i] = n[i].x;
                                acc[p][4 * i + 1] = n[i].y;
                                acc[p][4 * i + 2] = n[i].z;
                                acc[p][4 * i + 3] = n[i].w;
                            }
                            if constexpr (MODE == 1) {
#pragma unroll
                                for (int c = 0; c < DC; ++c) {
                                    const bf16x8 al = __builtin_bit_cast(bf16x8, Tl.a[c]);
                                    const bf16x8 ah = __builtin_bit_cast(bf16x8, T.a[c]);
                                    acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, P16.b[p][c], acc[p], 0, 0, 0);
                                    acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, P16lo.b[p][c], acc[p], 0, 0, 0);
                                    acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, P16.b[p][c], acc[p], 0, 0, 0);
                                }
                            } else {
#pragma unroll
                                for (int s = 0; s < 8 * DC; ++s)
                                    acc[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(T.a[s], P32.b[p][s], acc[p], 0, 0, 0);
                            }
                        }
                    }
                    consume(acc, need[half]);
                }
                store(tp);
            }
        };
        {
            auto no_store = [](int) {};
            if (ordered) {
                if constexpr (ROWS == 0) screen_pass1_tiles(MODE == 1 ? a.A : a.A16);
            } else if constexpr (MODE == 1) {
                if (a.lds_tiles)
                    screen_pass(BoolTag<true>{}, IntTag<1>{}, P16, a.A, pass1_consume, no_store);
                else
                    screen_pass(BoolTag<false>{}, IntTag<1>{}, P16, a.A, pass1_consume, no_store);
            } else {
                // FP32 mode: the BF16 tiles stream from global memory (the LDS
                // copy holds the FP32 tiles of pass 2)
                screen_pass(BoolTag<false>{}, IntTag<1>{}, P16, a.A16, pass1_consume, no_store);
            }
        }
        // thresholds: the jsel-th smallest of the point's 64 group minima (both
        // lanes' 32; negative values, from rounding, count as 0), as a key, or
        // (pair_select = 0: C above 32, jsel = ceil(C / 2)) the larger of the
        // two lanes' own jsel-th values.  Widened by both error bounds it screens both halves
        // in pass 2: the groups are disjoint, and a landmark counted by a BF16
        // group minimum has an exact key at most E16 above it and a pass-2 key
        // at most E2 above that, so the point has at least C candidates (jsel,
        // or 2 jsel); the certificate uses the pass-2 criterion itself.
        float tbase[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            int v0[16], v1[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                // approximate delta^2 as bit patterns; negative values (rounding)
                // become 0, and integer order is then float order
                v0[r] = max(__float_as_int(gmin[p][0][r] + xnp[p]), 0);
                v1[r] = max(__float_as_int(gmin[p][1][r] + xnp[p]), 0);
            }
            // (k known at compile time and C = k, the default)
            constexpr bool STATIC_J = KF == 1 && KP >= 8 && KP <= 24;
            if constexpr (KP == 1) {
                int t = v0[0];
#pragma unroll
                for (int r = 0; r < 16; ++r) t = min(t, min(v0[r], v1[r]));
                tbase[p] = __int_as_float(min(min(t, __shfl_xor(t, 32)), 0x7F7FFFFF));
            } else if (STATIC_J && a.pair_select && a.jsel == KP) {
                if constexpr (STATIC_J) tbase[p] = __int_as_float(min(select_pair_static<KP>(v0, v1), 0x7F7FFFFF));
            } else if (a.pair_select) {
                const int tl = min(select_pair_jth(v0, v1, a.jsel), 0x7F7FFFFF);  // +inf -> FLT_MAX
                tbase[p] = __int_as_float(tl);
            } else {
                const int tl = min(select_jth(v0, v1, a.jsel), 0x7F7FFFFF);
                const float own = __int_as_float(tl), oth = __int_as_float(__shfl_xor(tl, 32));
                tbase[p] = fmaxf(own, oth);
            }
        }

        // Pass-2 operands and their error bound e2.  BF16 mode splits the
        // point operand as x' = hi + lo + r (hi the pass-1 operand, lo = bf16(x'
        // - hi), both differences exact in FP32) and the landmark operand as
        // a = ah + al + ra likewise (from the preparation), and forms ah.hi +
        // al.hi + ah.lo, three BF16 products per element.  What it leaves out,
        // a.r - ra.r + al.lo + ra.x', is at most |r| (2 max|L - c| + max|ra|) +
        // max|al| |lo| + max|ra| |x'|; the FP32 accumulation of three chains of
        // d_pad products adds (6 d_pad + 16) u (|x'| + max|L - c|)^2 (the
        // single chain's allowance tripled).  |lo| and |r| are exact per point.
        // FP32 mode's FP32 operand is exact (e32).
        float e2[2];
        if constexpr (MODE == 1) {
            const float la = a.lmax[2], ra = a.lmax[3];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if constexpr (!SPLIT_EARLY) {
                    const int64_t si = pbase + 32 * p + i32;
                    const bool valid = si < a.n;
                    const float *xr = a.X + (valid ? slot_point<ROWS>(a, si) : 0) * a.ldx;
                    float lpart = 0.f, rpart = 0.f;
#pragma unroll
                    for (int c = 0; c < DC; ++c) {
                        float v[8];
                        centred8(xr, centL, a.d, c, h, valid, v);
                        // (opaque to the compiler, which would otherwise keep the first
                        // reading's unpacked high parts and remainders through pass 1:
                        // its tile loop then reloads 64 words a lane at 128-D)
                        u32x4 hw = __builtin_bit_cast(u32x4, P16.b[p][c]);
                        asm volatile("" : "+v"(hw));
                        P16.b[p][c] = __builtin_bit_cast(bf16x8, hw);
                        u32x4 lw;
#pragma unroll
                        for (int e = 0; e < 8; e += 2)
                            lw[e >> 1] = split_low(v[e] - bf16_lo(hw[e >> 1]), v[e + 1] - bf16_hi(hw[e >> 1]), lpart, rpart);
                        P16lo.b[p][c] = __builtin_bit_cast(bf16x8, lw);
                    }
                    nlo[p] = sqrtf(lpart + __shfl_xor(lpart, 32));
                    nre[p] = sqrtf(rpart + __shfl_xor(rpart, 32));
                }
                const float sx = sqrtf(xnp[p]);
                const float facc3 = (6.f * DP + 16.f) * U32 * (sx + lmax) * (sx + lmax);
                e2[p] = 1.01f * (nre[p] * (2.f * lmax + ra) + la * nlo[p] + ra * sx + facc3);
            }
        } else {
            e2[0] = e32[0];
            e2[1] = e32[1];
        }

        float tau[2], taucert[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            tau[p] = (tbase[p] >= FLT_MAX) ? FLT_MAX : (tbase[p] - xnp[p]) + (e16[p] + e2[p]);
            taucert[p] = tau[p];
        }

        // FP32 mode: the FP32 operand of pass 2 (the rows are still in cache)
        PointOperand<0, DC> P32;
        if constexpr (MODE == 0) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int64_t si = pbase + 32 * p + i32;
                const bool valid = si < a.n;
                const float *xr = a.X + (valid ? slot_point<ROWS>(a, si) : 0) * a.ldx;
#pragma unroll
                for (int c = 0; c < DC; ++c) {
                    float v[8];
                    centred8(xr, centL, a.d, c, h, valid, v);
#pragma unroll
                    for (int e = 0; e < 8; ++e) P32.b[p][8 * c + e] = v[e];
                }
            }
        }

        if constexpr (SPLIT_STASH) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int c = 0; c < DC; ++c) P16lo.b[p][c] = __builtin_bit_cast(bf16x8, stash[(p * DC + c) * 64]);
            wave_lds_fence();
        }

        // ---------------- pass 2: candidate bitmaps (key <= tau) into LDS.  The
        // sign of tau - key is shifted in (1 = not a candidate) and the word
        // complemented.  The two screen halves' words of a point and tile pair
        // sit side by side, bit-reversed, as one 64-bit word: bit 32 h + b is
        // position 64 tp + 2 b + h.  A mask per point marks the non-empty words.
        unsigned long long nonempty[2] = {0ull, 0ull};
        {
            unsigned word[2] = {0u, 0u};
            auto pass2_consume = [&](const f32x16 (&acc)[2], int) {
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        word[p] = __builtin_amdgcn_alignbit(word[p], __float_as_uint(tau[p] - acc[p][r]), 31);
            };
            auto pass2_store = [&](int tp) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const unsigned wd = ~word[p];
                    bitsL[((p * W + tp) * 32 + i32) * 2 + h] = __builtin_bitreverse32(wd);
                    nonempty[p] |= (unsigned long long)(wd != 0u) << tp;
                }
            };
            // a skipped half shifts in 16 "not a candidate" bits
            auto pass2_consume_skip = [&](const f32x16 (&acc)[2], const bool (&need)[2]) {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    if (need[p]) {
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            word[p] = __builtin_amdgcn_alignbit(word[p], __float_as_uint(tau[p] - acc[p][r]), 31);
                    } else {
                        word[p] = (word[p] << 16) | 0xFFFFu;
                    }
                }
            };
            if (ordered) {
                // tau + E16 + E2, rounded up, as an approximate delta^2
                unsigned thr16[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const float w = e16[p] + e2[p];
                    const float thr = (tau[p] + w) + 4.f * U32 * (fabsf(tau[p]) + w);
                    thr16[p] = (unsigned)max(__float_as_int(thr + xnp[p]), 0) >> 16;
                }
                if constexpr (ROWS == 0) screen_pass2_tiles(P32, pass2_consume_skip, pass2_store, thr16);
            } else if constexpr (MODE == 1) {
                if (a.lds_tiles)
                    screen_pass_split(BoolTag<true>{}, pass2_consume, pass2_store);
                else
                    screen_pass_split(BoolTag<false>{}, pass2_consume, pass2_store);
            } else {
                if (a.lds_tiles)
                    screen_pass(BoolTag<true>{}, IntTag<0>{}, P32, a.A, pass2_consume, pass2_store);
                else
                    screen_pass(BoolTag<false>{}, IntTag<0>{}, P32, a.A, pass2_consume, pass2_store);
            }
        }
        // Certificate bound per point: a non-candidate's exact distance^2
        // exceeds tau + |x - c|^2 - E, with E = e2 the error bound of the keys
        // pass 2 compared.
        if (h == 0) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const float E = e2[p];
                const float tc = taucert[p];
                float rhs = tc + xnp[p] - E;
                rhs -= 4.f * U32 * (fabsf(tc) + xnp[p] + E);
                certL[32 * p + i32] = (tc >= FLT_MAX) ? INFINITY : rhs;
            }
        }
        // masks of the points (p, i32): either screen half's word non-empty.  A
        // distance^2 is at most 2 (|x - c|^2 + max|L - c|^2).  Where that may leave
        // FP32 or is not a number, keys and bounds may be infinite or NaN, words may
        // hold the padding past the last landmark, and distances would pack to NaN
        // keys: such a point walks no candidate and is left to the exact path.
        // (Taking the padding out of the last word instead cost 0.8% at 1M x 32-D.)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const unsigned long long both = nonempty[p] | __shfl_xor(nonempty[p], 32);
            const bool within = fmaf(lmax, lmax, xnp[p]) < 0.125f * FLT_MAX;
            if (h == 0) maskL[32 * p + i32] = within ? both : 0ull;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // ---------------- phase B: one lane per point (lane l <-> slot pbase + l)
        const bool valid = pbase + lane < a.n;
        const int64_t pi = valid ? slot_point<ROWS>(a, pbase + lane) : 0;  // the point's own index
        const float cert_rhs = certL[lane];
        // The point's row.  ROWS = 1: in the lane's registers.  By quads (landmark
        // rows from memory): the four lanes of a quad rescore one candidate at a
        // time together, each on every fourth float4 of the rows, so x holds this
        // lane's pieces of its quad's four points: [4 c + 4 DC s ...] the
        // dimensions 16 c + 4 (lane mod 4) of the point of the quad's lane s.  A
        // load then covers 16 rows with 64 consecutive bytes each instead of 64
        // rows with 16: the kernel was bound by the L1's line accesses (0.92 a
        // clock at 1M x 48-D with 1024 landmarks, half of them the walk's).
        // Up to 16 dimensions a row is one line, and with the long lists (KP > 24)
        // the quads' moves cost more than they save: 200k points x 8-D, 600
        // landmarks, k = 28, 421 us by quads, 415 lane by lane; but 400k x 16-D, 1024
        // landmarks, k = 16, 250 and 255.
        float x[DP];
        constexpr bool QUADS = ROWS == 0 && (DC > 1 || KP <= 24);
        if constexpr (!QUADS) {
            const float *xr = a.X + (valid ? pi : 0) * a.ldx;
#pragma unroll
            for (int t = 0; t < DP / 4; ++t) {
                if (4 * t + 4 <= a.d) {
                    const Float4U v = reinterpret_cast<const Float4U *>(xr)[t];
                    x[4 * t] = v.x;
                    x[4 * t + 1] = v.y;
                    x[4 * t + 2] = v.z;
                    x[4 * t + 3] = v.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[4 * t + e] = 4 * t + e < a.d ? xr[4 * t + e] : 0.f;
                }
            }
        } else {
            const int pq = (int)(valid ? pi : 0);
            auto load_quad = [&](auto st) {
                constexpr int S = decltype(st)::value;
                const float *xr = a.X + (int64_t)quad_bcast<S>(pq) * a.ldx;
#pragma unroll
                for (int c = 0; c < DC; ++c) {
                    float *xc = x + 4 * (c + DC * S);
                    const int t0 = 16 * c + 4 * (lane & 3);
                    if (16 * c + 16 <= a.d) {
                        const Float4U v = *reinterpret_cast<const Float4U *>(xr + t0);
                        xc[0] = v.x;
                        xc[1] = v.y;
                        xc[2] = v.z;
                        xc[3] = v.w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) xc[e] = t0 + e < a.d ? xr[t0 + e] : 0.f;
                    }
                }
            };
            load_quad(IntTag<0>{});
            load_quad(IntTag<1>{});
            load_quad(IntTag<2>{});
            load_quad(IntTag<3>{});
        }
        double sk[KP];
#pragma unroll
        for (int q = 0; q < KP; ++q) sk[q] = INFINITY;
        double rej = INFINITY;
        int m = 0;
        // Each lane walks its own candidates across all its words (one candidate
        // per iteration), so the wave iterates max_l m_l times.  The next
        // non-empty word is read one word ahead.  The loop is wave-uniform (it
        // ends when no lane has a candidate left); a lane without one rescores
        // landmark 0 and inserts +inf, which leaves its list unchanged.  Keeping
        // the insertion out of divergent control flow keeps the list in place
        // in registers.
        {
            unsigned long long mk = valid ? maskL[lane] : 0ull;
            const unsigned long long *row = reinterpret_cast<const unsigned long long *>(bitsL) + h * W * 32 + i32;
            int ntp = 0, ctp = 0;
            unsigned long long nb = 0ull, b = 0ull;
            next_word(mk, row, nb, ntp);
            for (;;) {
                if (b == 0ull && nb != 0ull) {
                    b = nb;
                    ctp = ntp;
                    next_word(mk, row, nb, ntp);
                }
                const bool act = b != 0ull;
                if (__ballot(act) == 0ull) break;
                const int bit = act ? __builtin_ctzll(b) : 0;
                b &= b - 1ull;
                // bit 32 h + pos of a word of tile pair ctp: position 64 ctp + 2 pos + h
                const int j = act ? 64 * ctp + 2 * (bit & 31) + (bit >> 5) : 0;
                float acc = 0.f;
                auto add4 = [](float &sum, const float *xv, const float4 lv) {
                    const float e0 = xv[0] - lv.x, e1 = xv[1] - lv.y;
                    const float e2 = xv[2] - lv.z, e3 = xv[3] - lv.w;
                    sum = fmaf(e0, e0, sum);
                    sum = fmaf(e1, e1, sum);
                    sum = fmaf(e2, e2, sum);
                    sum = fmaf(e3, e3, sum);
                };
                // rows from the block's LDS copy, or by quads from memory
                if constexpr (!QUADS) {
                    const float4 *Lr = ROWS ? reinterpret_cast<const float4 *>(rowsL + row_offset<RS>(j))
                                            : reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(a.Lpad) + row_offset<4 * DP>(j));
                    // four partial sums joined as the quads join theirs, so that a
                    // distance has the same bits wherever the rows lie
                    float sum[4] = {0.f, 0.f, 0.f, 0.f};
                    // (Four reads in flight: left to itself the compiler issues and
                    // awaits them one by one here; 20k points x 64-D, 400 landmarks, k =
                    // 16, 92 us a call, 86 so, and no less with eight.  Beyond 64
                    // dimensions it takes registers from the row: 200k x 128-D, 100
                    // landmarks, k = 24, 585 us so, 332 without.)
#pragma unroll
                    for (int c = 0; c < DC; ++c) {
                        float4 lv[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) lv[q] = Lr[4 * c + q];
                        if constexpr (DC <= 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int q = 0; q < 4; ++q) add4(sum[q], x + 4 * (4 * c + q), lv[q]);
                    }
                    acc = (sum[0] + sum[1]) + (sum[2] + sum[3]);
                } else {
                    const char *base = reinterpret_cast<const char *>(a.Lpad);
                    const unsigned off = mul24((unsigned)j, 4u * DP);
                    const unsigned o[4] = {(unsigned)quad_bcast<0>((int)off) + 16u * (lane & 3),
                                           (unsigned)quad_bcast<1>((int)off) + 16u * (lane & 3),
                                           (unsigned)quad_bcast<2>((int)off) + 16u * (lane & 3),
                                           (unsigned)quad_bcast<3>((int)off) + 16u * (lane & 3)};
                    // The loads go through the four candidates' rows 64 bytes at
                    // a time, so that a line's second half follows its first
                    // after 64 other accesses: an access to a line still on its
                    // way stalls the L1 (row by row, its pending-stall cycles
                    // doubled and the fused kernel took 1.010 ms at 1M x 48-D;
                    // in this order 0.790 ms, lane by lane 0.896 ms, and at 10M
                    // x 64-D 8.25 against 10.26 ms).
                    float sum[4] = {0.f, 0.f, 0.f, 0.f};
                    // chunks in flight, 16 registers each (200k x 128-D, 1024
                    // landmarks, k = 16: all 8 at once 707 us, 4 and 4 528)
                    constexpr int CH = DC <= 4 ? DC : 4;
#pragma unroll
                    for (int c0 = 0; c0 < DC; c0 += CH) {
                        float4 lv[CH][4];
#pragma unroll
                        for (int c = 0; c < CH; ++c)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (c0 + c < DC)
                                    lv[c][q] = *reinterpret_cast<const float4 *>(base + (size_t)(o[q] + 64u * (c0 + c)));
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int c = 0; c < CH; ++c)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (c0 + c < DC) add4(sum[q], x + 4 * (c0 + c + DC * q), lv[c][q]);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float t = quad_sum(sum[q]);
                        acc = (lane & 3) == q ? t : acc;
                    }
                }
                // keys carry the landmark index (ties break on it), not the position
                insert_sorted<KP>(sk, rej, act ? pack_key(acc, permL[j]) : (double)INFINITY);
                m += act ? 1 : 0;
            }
        }
        __builtin_amdgcn_wave_barrier();

        // k-th and (k+1)-th rescored distances
        float d2k = 0.f, d2k1 = INFINITY;
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            if (q == a.k - 1) d2k = key_d2(sk[q]);
            if (q == a.k) d2k1 = key_d2(sk[q]);
        }
        if (a.k >= KP) d2k1 = (rej < INFINITY) ? key_d2(rej) : INFINITY;
        const float thr = kth_bound(m >= a.k ? d2k : INFINITY, DP);

        unsigned reason = 0;
        {
            const bool cert = d2k * (1.f + (DP + 3) * U32) < cert_rhs;
            if (!cert || m < a.k) reason |= R_UNCERT;
            // two rescored values are ordered correctly when their gap exceeds the sum
            // of their rounding bounds, (d_pad + 3) u each
            if (m > a.k && d2k1 - d2k <= 2.f * (DP + 3) * U32 * d2k1) reason |= R_NEARTIE;
            // When the caller asked for the neighbour list (its first entry is the
            // nearest landmark of the landmark update), adjacent entries closer
            // than the rounding bound are ranked again, so the list is ordered
            // by exact distance.  (The serving cache keeps the fast path's own
            // order, which is what a fresh projection uses.)
            if (a.knn_exact_order) {
                float prev = key_d2(sk[0]);
#pragma unroll
                for (int q = 1; q < KP; ++q) {
                    const float cur = key_d2(sk[q]);
                    if (q < a.k && q < m && cur - prev <= 2.f * (DP + 3) * U32 * cur) reason |= R_ORDER;
                    prev = cur;
                }
            }
        }

        // FP64 distances for small cutoff weights (k <= 8 only), while the
        // point's row is in registers; landmark rows from the LDS copy or the
        // padded array (zero past d in both).  A weight's FP32 error matters when
        // its pairs compete with gravity alone in some direction, which needs
        // the other neighbours' pairs to be rank-deficient in 2-D: plausible
        // for a few neighbours; with more, the strong pairs fix both directions
        // or the system is flagged as ill-conditioned.  At k <= 16 the code
        // alone cost 8% of this kernel (register pressure), used or not.
        float cref[N_REFINE] = {};
        int nref = 0;
        if constexpr (KP <= 8 && KP > 1) {
            if (!a.knn_only) {
                // the walk's sums in FP64: four parts, joined as the quads join theirs.
                // Rows of more than 64 dimensions are read again from memory, lane by
                // lane (held until here they cost registers).  Below, quads read them
                // as in the walk: lane by lane, 200k uniform points x 64-D, 1024
                // landmarks, k = 8 took 404 us a call, now 332.
                const float *xr = a.X + (valid ? pi : 0) * a.ldx;
                auto d2x = [&](int jl) -> double {
                    const unsigned pos = iposL[jl];
                    double sum[4] = {0.0, 0.0, 0.0, 0.0};
                    auto add4 = [](double &acc, const float *xv, const float4 lv) {
                        const double e0 = (double)xv[0] - (double)lv.x, e1 = (double)xv[1] - (double)lv.y;
                        const double e2 = (double)xv[2] - (double)lv.z, e3 = (double)xv[3] - (double)lv.w;
                        acc = fma(e0, e0, acc);
                        acc = fma(e1, e1, acc);
                        acc = fma(e2, e2, acc);
                        acc = fma(e3, e3, acc);
                    };
                    if constexpr (QUADS && DC <= 4) {
                        const char *base = reinterpret_cast<const char *>(a.Lpad);
                        const int off = (int)mul24(pos, 4u * DP);
                        const unsigned lo16 = 16u * (lane & 3);
                        const unsigned o[4] = {(unsigned)quad_bcast<0>(off) + lo16, (unsigned)quad_bcast<1>(off) + lo16,
                                               (unsigned)quad_bcast<2>(off) + lo16, (unsigned)quad_bcast<3>(off) + lo16};
#pragma unroll
                        for (int c = 0; c < DC; ++c) {
                            float4 lv[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                lv[q] = *reinterpret_cast<const float4 *>(base + (size_t)(o[q] + 64u * c));
#pragma unroll
                            for (int q = 0; q < 4; ++q) add4(sum[q], x + 4 * (c + DC * q), lv[q]);
                        }
                        double own = 0.0;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const double t = quad_sum64(sum[q]);
                            own = (lane & 3) == q ? t : own;
                        }
                        return own;
                    }
                    const float4 *Lr = ROWS ? reinterpret_cast<const float4 *>(rowsL + row_offset<RS>(pos))
                                            : reinterpret_cast<const float4 *>(a.Lpad + (size_t)pos * DP);
                    if constexpr (DC <= 4) {
#pragma unroll
                        for (int q = 0; q < DP / 4; ++q) add4(sum[q & 3], x + 4 * q, Lr[q]);
                    } else {
#pragma unroll 4
                        for (int q = 0; q < DP / 4; ++q) {
                            float xv[4];
                            if (4 * q + 4 <= a.d) {
                                const Float4U u = reinterpret_cast<const Float4U *>(xr)[q];
                                xv[0] = u.x;
                                xv[1] = u.y;
                                xv[2] = u.z;
                                xv[3] = u.w;
                            } else {
#pragma unroll
                                for (int e = 0; e < 4; ++e) xv[e] = 4 * q + e < a.d ? xr[4 * q + e] : 0.f;
                            }
                            add4(sum[q & 3], xv, Lr[q]);
                        }
                    }
                    return (sum[0] + sum[1]) + (sum[2] + sum[3]);
                };
                reason |= refine_cutoffs<KP>(a, sk, valid, d2x, cref, nref);
            }
        }

        // knn outputs (the exact path rewrites those of uncertified / near-tie points)
        if (valid && a.knn_mark) a.knn_mark[pi] = (reason & (R_UNCERT | R_NEARTIE)) ? 1 : 0;
        if (valid && (a.knn_idx || a.knn_d2)) {
#pragma unroll
            for (int q = 0; q < KP; ++q) {
                if (q < a.k) {
                    if (a.knn_idx) a.knn_idx[pi * a.k + q] = key_idx(sk[q]);
                    if (a.knn_d2) a.knn_d2[pi * a.k + q] = key_d2(sk[q]);
                }
            }
        }

        if (KP > 1 && !a.knn_only) {
            __builtin_amdgcn_wave_barrier();
            if constexpr (KP > 1) reason = project_point<KP>(a, sk, lane, valid, pi, reason, nbD2, nbS, nbI, iposL, cref, nref);
        }
        if (valid && reason) list_point(a, pi, reason, thr);
        st_cand += valid ? (unsigned long long)m : 0ull;
    }
    // wave-level totals
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) st_cand += __shfl_xor(st_cand, o);
    if (lane == 0 && st_cand) atomicAdd(&a.counters[C_CAND], st_cand);
}

}  // namespace esom
