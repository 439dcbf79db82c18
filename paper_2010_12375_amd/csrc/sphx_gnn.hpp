// sphx_gnn.hpp -- HIP kernels (gfx950) of the message-passing surrogate on
// the SPH neighbour graph: features from the frozen configuration, BF16 MFMA
// matrix products with FP32 accumulation, edge messages summed per particle,
// the backward pass, Adam and the surrogate's state update.
//
// The network (hidden width 64, 3 layers) predicts each fluid particle's
// mean acceleration and density rate over the next two advection steps:
//   H = relu(F Wn + bn),  E0 = relu(G We + be)
//   layer: P = H Wa + bm, Q = H Wb, R = E0 Wc; m_e = relu(P_i + Q_j + R_e)
//          (a wall edge takes the learned vector qw in place of Q_j);
//          A_i = sum_e m_e;  H <- H + relu([H | A] Wu + bu)
//   Y = relu(H Wo1 + bo1) Wo2 + bo2 = (a_x/g, a_y/g, 1000 Drho h / (rho0 u_ref))
// Node rows are the fluid slots of the batch layout (padding slots carry
// zeros); edge rows are, per particle, its inner then its contact entries in
// list order (CSR by particle). Activations are FP32; every matrix-product
// operand is rounded to bfloat16 (nearest, ties to even) as it is loaded into
// an MFMA fragment, and the products accumulate in FP32. The last product
// (D1 Wo2, 64 -> 3) runs in FP32 on the vector units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sphx_device.hpp"

namespace sphx {
namespace gnn {

constexpr int HID = 64;
constexpr int FPAD = 32;   // padded encoder input width
constexpr int EFEAT = 8;   // edge features used
constexpr int NOUT = 3;
constexpr unsigned ROW_BYTES = HID * sizeof(float);  // of an FP32 row
constexpr int WALL_EDGE = -1;  // edst < 0: wall edge, wall index -1 - edst

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest, ties to even (finite inputs)
__device__ __forceinline__ uint32_t bf16_bits(float x)
{
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// The same for two floats in one instruction (v_cvt_pk_bf16_f32): lo in the
// low half. The bit arithmetic above costs nine.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi)
{
    const bf16x2 b = __builtin_convertvector(f32x2{lo, hi}, bf16x2);
    return __builtin_bit_cast(uint32_t, b);
}

union Frag {
    bf16x8 v;
    uint32_t u[4];
    uint4 q;
};

// Eight consecutive floats rounded into an MFMA operand fragment.
__device__ __forceinline__ bf16x8 frag_from_f32(const float* p, bool ok)
{
    Frag f;
    if (ok) {
        const float4 a = *(const float4*)p;
        const float4 b = *(const float4*)(p + 4);
        f.u[0] = bf16_pair(a.x, a.y);
        f.u[1] = bf16_pair(a.z, a.w);
        f.u[2] = bf16_pair(b.x, b.y);
        f.u[3] = bf16_pair(b.z, b.w);
    } else {
        f.q = make_uint4(0u, 0u, 0u, 0u);
    }
    return f.v;
}

__device__ __forceinline__ bf16x8 frag_from_bf16(const uint16_t* p)
{
    Frag f;
    f.q = *(const uint4*)p;
    return f.v;
}

// ---------------------------------------------------------------------
// Matrix product with a 64-wide output:
//   C[M x 64] = epi(A[M x K] B),  A FP32 rows of stride lda, B given as
//   Bt = B^T in bf16 [64 x K] (row-major, K contiguous).
// One wavefront computes 16 rows (four 16x16 tiles) with
// v_mfma_f32_16x16x32_bf16: lane l supplies row (l mod 16) of A and column
// (l mod 16) of B at the 8 K positions 8 (l div 16) + 0..7 of each 32-wide K
// step (the same positions for A and B, so the pairing is exact), and holds
// output rows 4 (l div 16) + 0..3 of column (l mod 16).
enum Epi : int {
    EPI_STORE = 0,  // C = acc + bias
    EPI_RELU = 1,   // C = relu(acc + bias)
    EPI_ACCUM = 2,  // C += acc
    EPI_RESID = 3,  // C2 = acc + bias (pre-activation); C += relu(acc + bias)
};

template <int K, int EPI>
__global__ __launch_bounds__(256) void k_gemm64(int M, const float* __restrict__ A, int lda,
                                                const uint16_t* __restrict__ Bt, const float* __restrict__ bias,
                                                float* __restrict__ C, int ldc, float* __restrict__ C2, int ldc2)
{
    static_assert(K % 32 == 0, "K must be a multiple of 32");
    const int lane = threadIdx.x & 63;
    const int m0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
    if (m0 >= M) return;
    const int r = lane & 15, g = lane >> 4;
    f32x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ra = m0 + r;
    const bool ok = ra < M;
#pragma unroll
    for (int ks = 0; ks < K; ks += 32) {
        const bf16x8 a = frag_from_f32(A + (size_t)(ok ? ra : 0) * lda + ks + 8 * g, ok);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bf16x8 b = frag_from_bf16(Bt + (size_t)(16 * t + r) * K + ks + 8 * g);
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int col = 16 * t + r;
        const float bv = bias ? bias[col] : 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = m0 + 4 * g + q;
            if (row >= M) continue;
            const float v = acc[t][q];
            float* c = C + (size_t)row * ldc + col;
            if constexpr (EPI == EPI_STORE) {
                *c = v + bv;
            } else if constexpr (EPI == EPI_RELU) {
                *c = fmaxf(v + bv, 0.f);
            } else if constexpr (EPI == EPI_ACCUM) {
                *c = *c + v;
            } else {
                const float z = v + bv;
                C2[(size_t)row * ldc2 + col] = z;
                *c = *c + fmaxf(z, 0.f);
            }
        }
    }
}

// The lane's column of a row of 64 floats, the row given by a uniform key. Up
// to ROWS32 nodes the key is the row's byte offset and the row is read with a
// buffer load, which takes the offset from a scalar register as it is; beyond
// (BIG) offsets do not fit 32 bits: the key is the row's number and the
// address a 64-bit product.
constexpr int ROWS32 = (1 << 24) - 2;  // with the two special rows of Q
template <bool BIG> struct Rows;
template <> struct Rows<false> {
    __amdgpu_buffer_rsrc_t p;
    __device__ __forceinline__ Rows(const float* a, int n)
        : p(__builtin_amdgcn_make_buffer_rsrc((void*)a, 0, (int)((unsigned)n * ROW_BYTES), 0x00020000))
    {
    }
    static __host__ __device__ __forceinline__ int key(int row) { return (int)((unsigned)row * ROW_BYTES); }
    __device__ __forceinline__ float at(int k, int lane) const
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(p, lane * (int)sizeof(float), k, 0));
    }
};
template <> struct Rows<true> {
    const float* p;
    __device__ __forceinline__ Rows(const float* a, int) : p(a) {}
    static __host__ __device__ __forceinline__ int key(int row) { return row; }
    __device__ __forceinline__ float at(int k, int lane) const { return p[(size_t)(unsigned)k * HID + lane]; }
};

// ---------------------------------------------------------------------
// Weight gradient dW[KIN x 64] = X^T dZ over M rows, split over blocks of
// `rows` rows each (partials summed later in a fixed order), and with `bpart`
// the column sums of dZ (bias gradient) in FP32, row by row. Each step takes
// WROWS rows: a wavefront loads 16 of them with one lane per column, so that
// a lane holds 16 rows of its column, which it rounds to bf16 and writes as
// whole 16-byte pieces of the transposed LDS arrays; the next step's loads
// are in flight while wavefront w computes output column tile w for all
// KIN/16 row tiles. Bound by HBM: X and dZ are read once. (A load, a
// conversion and a 2-byte LDS write per element, and the bias from a second
// serial read of dZ: 100 us for 205k rows of 64 + 64 columns, 21 us of
// traffic.)
constexpr int WROWS = 64;      // rows per step
constexpr int WPAD = WROWS + 8;

// Round the 16 rows of a lane's column and store them from row `at`.
__device__ __forceinline__ void store_rows16(uint16_t* p, const float v[16])
{
    uint4 a, b;
    a.x = bf16_pair(v[0], v[1]);
    a.y = bf16_pair(v[2], v[3]);
    a.z = bf16_pair(v[4], v[5]);
    a.w = bf16_pair(v[6], v[7]);
    b.x = bf16_pair(v[8], v[9]);
    b.y = bf16_pair(v[10], v[11]);
    b.z = bf16_pair(v[12], v[13]);
    b.w = bf16_pair(v[14], v[15]);
    *(uint4*)p = a;
    *(uint4*)(p + 8) = b;
}

// acc[t] += X^T dZ of one staged step: rows of Xs are X's columns (TM tiles
// of 16), Zs's are dZ's, both bf16 with WROWS rows contiguous.
template <int TM>
__device__ __forceinline__ void wgrad_step(const uint16_t (*Xs)[WPAD], const uint16_t (*Zs)[WPAD], int w, int r, int g,
                                           f32x4 acc[TM])
{
#pragma unroll
    for (int k = 0; k < WROWS; k += 32) {
        const bf16x8 fb = frag_from_bf16(&Zs[16 * w + r][k + 8 * g]);
#pragma unroll
        for (int t = 0; t < TM; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_bf16(&Xs[16 * t + r][k + 8 * g]), fb, acc[t], 0, 0, 0);
    }
}

template <int KIN>
__global__ __launch_bounds__(256) void k_wgrad(int M, int rows, const float* __restrict__ X, int ldx,
                                               const float* __restrict__ dZ, int ldz, float* __restrict__ part,
                                               float* __restrict__ bpart)
{
    constexpr int TM = KIN / 16;
    constexpr int XL = KIN / 4;  // X values per lane and step (16 rows x KIN columns over 64 lanes)
    __shared__ __align__(16) uint16_t Xs[KIN][WPAD];
    __shared__ __align__(16) uint16_t Zs[HID][WPAD];
    __shared__ float Zf[WROWS][HID];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    f32x4 acc[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    const int r0 = blockIdx.x * rows;
    const int r1 = min(r0 + rows, M);
    float z[16], x[XL];
    auto load = [&](int rb) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int row = rb + 16 * w + q;
            z[q] = row < r1 ? dZ[(size_t)row * ldz + lane] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < XL; ++q) {
            // KIN = 32: half a wavefront per row, rows q and q + 8
            const int row = rb + 16 * w + (KIN == 32 ? 8 * (lane >> 5) + q : q % 16);
            const int col = KIN == 32 ? (lane & 31) : lane + 64 * (q / 16);
            x[q] = row < r1 ? X[(size_t)row * ldx + col] : 0.f;
        }
    };
    load(r0);
    for (int rb = r0; rb < r1; rb += WROWS) {
        store_rows16(&Zs[lane][16 * w], z);
        if constexpr (KIN == 32) {
            *(uint4*)&Xs[lane & 31][16 * w + 8 * (lane >> 5)] = make_uint4(
                bf16_pair(x[0], x[1]), bf16_pair(x[2], x[3]), bf16_pair(x[4], x[5]), bf16_pair(x[6], x[7]));
        } else {
#pragma unroll
            for (int c = 0; c < KIN / 64; ++c) store_rows16(&Xs[lane + 64 * c][16 * w], x + 16 * c);
        }
        if (bpart)
#pragma unroll
            for (int q = 0; q < 16; ++q) Zf[16 * w + q][lane] = z[q];
        __syncthreads();
        if (rb + WROWS < r1) load(rb + WROWS);
        wgrad_step<TM>(Xs, Zs, w, r, g, acc);
        if (bpart && threadIdx.x < HID) {
            const int n = min(WROWS, r1 - rb);
#pragma unroll 16
            for (int q = 0; q < n; ++q) bsum += Zf[q][threadIdx.x];
        }
        __syncthreads();
    }
    float* out = part + (size_t)blockIdx.x * KIN * HID;
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(size_t)(16 * t + 4 * g + q) * HID + 16 * w + r] = acc[t][q];
    if (bpart && threadIdx.x < HID) bpart[(size_t)blockIdx.x * HID + threadIdx.x] = bsum;
}

// out[j] = sum over b of part[b][j], b ascending (deterministic), for two
// arrays in one launch: blocks below nblk1 the first, the rest the second.
// A block takes 16 columns: 256 rows at a time go through LDS with 16 loads
// in flight per thread, then one lane per column adds them in order. (One
// thread per column reading its column row by row waited out a memory round
// trip per few rows: 185 us for 1024 x 4096, 17 MB.)
constexpr int RCOLS = 16;
__global__ __launch_bounds__(256) void k_reduce_parts(int nb, int nblk1, int len, const float* __restrict__ part,
                                                      float* __restrict__ out, int len2,
                                                      const float* __restrict__ part2, float* __restrict__ out2)
{
    __shared__ float sh[256][RCOLS + 1];
    int bx = blockIdx.x;
    if (bx >= nblk1) {
        bx -= nblk1;
        len = len2;
        part = part2;
        out = out2;
    }
    const int c = threadIdx.x % RCOLS, rr = threadIdx.x / RCOLS;
    const int j = bx * RCOLS + c;
    float s = 0.f;
    for (int b0 = 0; b0 < nb; b0 += 256) {
        float v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int b = b0 + rr + 16 * q;
            v[q] = b < nb && j < len ? part[(size_t)b * len + j] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) sh[rr + 16 * q][c] = v[q];
        __syncthreads();
        if (threadIdx.x < RCOLS) {
            const int n = min(256, nb - b0);
#pragma unroll 16
            for (int b = 0; b < n; ++b) s += sh[b][c];
        }
        __syncthreads();
    }
    if (threadIdx.x < RCOLS && j < len) out[j] = s;
}

// Column sums of a [M x 64] FP32 matrix in row blocks (partials).
__global__ __launch_bounds__(64) void k_colsum64(int M, int rows, const float* __restrict__ A, int lda,
                                                 float* __restrict__ part)
{
    const int r0 = blockIdx.x * rows, r1 = min(r0 + rows, M);
    float s = 0.f;
    int r = r0;
    for (; r + 32 <= r1; r += 32) {  // 32 loads in flight
        float v[32];
#pragma unroll
        for (int q = 0; q < 32; ++q) v[q] = A[(size_t)(r + q) * lda + threadIdx.x];
#pragma unroll
        for (int q = 0; q < 32; ++q) s += v[q];
    }
    for (; r < r1; ++r) s += A[(size_t)r * lda + threadIdx.x];
    part[(size_t)blockIdx.x * HID + threadIdx.x] = s;
}

// ---------------------------------------------------------------------
// Graph: per-slot edge counts, then (after a scan) the CSR edges with their
// features, the reverse of every inner edge, and the node features.

template <typename real>
__global__ __launch_bounds__(BLOCK) void k_gnn_count(const KP<real>* __restrict__ Pt, const int32_t* __restrict__ tcase,
                                                     int ntiles, const int32_t* __restrict__ ncnt,
                                                     const int32_t* __restrict__ wcnt, int32_t* __restrict__ ecount)
{
    const int tile = wave_tile();
    if (tile >= ntiles) return;
    const KP<real>& P = Pt[tcase[tile]];
    const int i = tile * TILE + (threadIdx.x & 63);
    ecount[i] = i < P.fbase + P.nf ? ncnt[i] + wcnt[i] : 0;
}

__device__ __forceinline__ float wendland_ratio(float q)
{
    const float s = fmaxf(1.f - 0.5f * q, 0.f);
    return s * s * s * s * (1.f + 2.f * q);
}

// Constants of a case's features.
struct FeatScale {
    float inv_u, inv_h, gx, gy, inv_pscale, c2, rho0;
};
template <typename real>
__device__ __forceinline__ FeatScale feat_scale(const KP<real>& P)
{
    FeatScale c;
    c.inv_u = (float)(1.0 / P.u_ref);
    c.inv_h = (float)P.inv_h;
    c.gx = (float)P.g[0];
    c.gy = (float)P.g[1];
    const float gmag = sqrtf(c.gx * c.gx + c.gy * c.gy + (float)P.g[2] * (float)P.g[2]);
    c.inv_pscale = 1.f / ((float)P.rho0 * gmag) * c.inv_h;
    c.c2 = (float)P.c2;
    c.rho0 = (float)P.rho0;
    return c;
}

// The EFEAT features of one edge (x_j - x_i = -(dx, dy)).
__device__ __forceinline__ void edge_features(const FeatScale& c, float dx, float dy, float dvx, float dvy, float wall,
                                              float dpres, float f[EFEAT])
{
    const float rr = sqrtf(dx * dx + dy * dy);
    f[0] = -dx * c.inv_h;
    f[1] = -dy * c.inv_h;
    f[2] = rr * c.inv_h;
    f[3] = dvx * c.inv_u;
    f[4] = dvy * c.inv_u;
    f[5] = wendland_ratio(rr * c.inv_h);
    f[6] = wall;
    f[7] = dpres * c.inv_pscale;
}

// The edges in CSR order with their features: EL lanes per slot, each taking
// every EL-th entry. Edge features (x_j - x_i)/h, r/h, (v_j - v_i)/u_ref,
// W(r)/W(0), wall flag, pressure difference (p_j - p_i)/(rho0 |g| h) (for a
// wall the one-sided wall state, p_w - p_i = rho_i g.(x_w - x_i)), taken in
// FP32 from the density deviations before any rounding; node features
// v/u_ref, (rho - rho0)/(0.01 rho0), inner and contact counts / 32 and / 16
// (2D).
//
// G rows hold `ldg` floats: EFEAT (the features alone) or FPAD (zero-padded,
// for the unfused encoder product). esrc receives the key (Rows) of the
// row of each edge's particle; the reverse edges (erev, for the
// backward of Q_j) are searched only when erev is given. (One thread per slot
// left 3 200 wavefronts with a serial search each: 700 us at 205k nodes.)
constexpr int EL = 8;
template <typename real, int T, bool BIG>
__global__ __launch_bounds__(BLOCK) void k_gnn_edges(
    const KP<real>* __restrict__ Pt, const int32_t* __restrict__ tcase, int N, const int32_t* __restrict__ eoff,
    const uint32_t* __restrict__ nbr, const int32_t* __restrict__ ncnt, const uint32_t* __restrict__ wnb,
    const int32_t* __restrict__ wcnt, const R2<real>* __restrict__ geo, const R2<real>* __restrict__ wgeo,
    const R4<real>* __restrict__ st, int32_t* __restrict__ edst, int32_t* __restrict__ erev,
    int32_t* __restrict__ esrc, float* __restrict__ G, int ldg, float* __restrict__ F)
{
    const int i = (blockIdx.x * BLOCK + threadIdx.x) / EL, l = threadIdx.x % EL;
    if (i >= N) return;
    const KP<real>& P = Pt[tcase[i / TILE]];
    float4* f = (float4*)(F + (size_t)i * FPAD);
    const bool used = i < P.fbase + P.nf;
    const R4<real> si = used ? st[i] : R4<real>{};
    const float devi = (float)si.z;
    const float vix = (float)si.x, viy = (float)si.y;
    const int nin = used ? ncnt[i] : 0, nwl = used ? wcnt[i] : 0;
    const FeatScale c = feat_scale(P);
    // node features: FPAD floats, four per lane
    static_assert(FPAD == 4 * EL, "one float4 of node features per lane");
    float4 fv = make_float4(0.f, 0.f, 0.f, 0.f);
    if (used && l == 0)
        fv = make_float4(vix * c.inv_u, viy * c.inv_u, (float)si.z / (0.01f * (float)P.rho0), (float)nin / 32.f);
    if (used && l == 1) fv.x = (float)nwl / 16.f;
    f[l] = fv;
    if (!used) return;
    const R2<real> oi = geo[i];
    const int e0 = eoff[i];
    auto edge = [&](int e, float dx, float dy, float dvx, float dvy, float wall, float dpres) {
        float q[EFEAT];
        edge_features(c, dx, dy, dvx, dvy, wall, dpres, q);
        float4* gr = (float4*)(G + (size_t)e * ldg);
        gr[0] = make_float4(q[0], q[1], q[2], q[3]);
        gr[1] = make_float4(q[4], q[5], q[6], q[7]);
        for (int k = EFEAT / 4; k < ldg / 4; ++k) gr[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        esrc[e] = Rows<BIG>::key(i);
    };
    for (int k = l; k < nin; k += EL) {
        const int e = e0 + k;
        const uint32_t ent = nbr[ell_at<T>(i, k, P.maxn)];
        const int j = (int)(ent & NBR_MASK);
        const uint32_t code = ent >> NBR_SHIFT;
        const R2<real> oj = geo[j];
        const float dx = (float)((oi.x - oj.x) - (real)((int)(code & 3u) - 1) * P.L[0]);
        const float dy = (float)((oi.y - oj.y) - (real)((int)((code >> 2) & 3u) - 1) * P.L[1]);
        const R4<real> sj = st[j];
        edge(e, dx, dy, (float)sj.x - vix, (float)sj.y - viy, 0.f, c.c2 * ((float)sj.z - devi));
        edst[e] = j;
        if (erev) {
            // the reverse edge: i in the inner list of j (the lists are symmetric)
            int rv = -1;
            const int nj = ncnt[j];
            for (int kk = 0; kk < nj; ++kk)
                if ((int)(nbr[ell_at<T>(j, kk, P.maxn)] & NBR_MASK) == i) {
                    rv = eoff[j] + kk;
                    break;
                }
            erev[e] = rv;
        }
    }
    for (int k = l; k < nwl; k += EL) {
        const int e = e0 + nin + k;
        const uint32_t ent = wnb[ell_at<T>(i, k, P.maxw)];
        const int wj = (int)(ent & NBR_MASK);
        const uint32_t code = ent >> NBR_SHIFT;
        const R2<real> ow = wgeo[wj];
        const float dx = (float)((oi.x - ow.x) - (real)((int)(code & 3u) - 1) * P.L[0]);
        const float dy = (float)((oi.y - ow.y) - (real)((int)((code >> 2) & 3u) - 1) * P.L[1]);
        edge(e, dx, dy, -vix, -viy, 1.f, (c.rho0 + devi) * (c.gx * -dx + c.gy * -dy));
        edst[e] = -1 - wj;
        if (erev) erev[e] = -1;
    }
}

// ---------------------------------------------------------------------
// Messages of the unfused layer (sphx_gnn_profile's comparison): one
// wavefront per node row, lane = feature,
//   A_i = sum_e relu(P_i + (Q_j | qw) + R_e) -> X[i][64 + f]
__global__ __launch_bounds__(256) void k_gnn_msg(int N, const int32_t* __restrict__ eoff,
                                                 const int32_t* __restrict__ edst, const float* __restrict__ P,
                                                 const float* __restrict__ Q, const float* __restrict__ R,
                                                 const float* __restrict__ qw, float* __restrict__ X)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= N) return;
    const int f = threadIdx.x & 63;
    const float p = P[(size_t)i * HID + f];
    const float q0 = qw[f];
    float acc = 0.f;
    for (int e = eoff[i]; e < eoff[i + 1]; ++e) {
        const int d = edst[e];
        const float pre = p + (d >= 0 ? Q[(size_t)d * HID + f] : q0) + R[(size_t)e * HID + f];
        acc += fmaxf(pre, 0.f);
    }
    X[(size_t)i * 2 * HID + HID + f] = acc;
}

// The forward pass is four launches, straight from the neighbour lists: the
// node encoder (with layer 0's P and Q) and one kernel per layer (with the
// next layer's P and Q, or the decoder). Nothing per edge reaches HBM in
// inference, and no edge count is needed on the host; a training pass keeps
// one bit per message (its sign, for the backward pass) and the node arrays.
// Every value is rounded where and summed in the order in which the unfused
// products and sums round and sum it, so the two agree bit for bit.

// Rows N and N + 1 of a Q array: the learned vector that stands for Q_j at a
// wall edge, and one of -inf, whose message relu(P_i - inf + R_e) is 0
// whatever P_i and R_e hold, NaN included (a tile row without an edge). Edges
// then differ only in the row they read.
__device__ __forceinline__ void special_rows(float* __restrict__ Q, int N, const float* __restrict__ qw)
{
    if (blockIdx.x != 0 || threadIdx.x >= HID) return;
    Q[(size_t)N * HID + threadIdx.x] = qw[threadIdx.x];
    Q[(size_t)(N + 1) * HID + threadIdx.x] = -__builtin_inff();
}

// Node encoder H = relu(F Wn + bn), P = H Wa + bm, Q = H Wb of 16 nodes per
// wavefront; the features are taken from the particle state in registers
// (only lanes with g = 0 hold nonzero inputs).
template <typename real>
__global__ __launch_bounds__(256) void k_gnn_encode(
    const KP<real>* __restrict__ Pt, const int32_t* __restrict__ tcase, int N, const int32_t* __restrict__ ncnt,
    const int32_t* __restrict__ wcnt, const R4<real>* __restrict__ st, const uint16_t* __restrict__ WnT,
    const float* __restrict__ bn, const uint16_t* __restrict__ WaT, const float* __restrict__ bm,
    const uint16_t* __restrict__ WbT, const float* __restrict__ qw, float* __restrict__ H, int ldh,
    float* __restrict__ Pm, float* __restrict__ Qm)
{
    special_rows(Qm, N, qw);
    __shared__ __align__(16) uint16_t Hs[4][16][HID + 8];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int m0 = (blockIdx.x * 4 + wv) * 16;
    if (m0 >= N) return;  // N is a multiple of TILE: whole groups of 16 nodes
    const KP<real>& P = Pt[tcase[m0 / TILE]];
    const int i = m0 + r;
    Frag f;
    f.q = make_uint4(0u, 0u, 0u, 0u);
    if (g == 0 && i < P.fbase + P.nf) {
        const float inv_u = (float)(1.0 / P.u_ref);
        const R4<real> si = st[i];
        f.u[0] = bf16_pair((float)si.x * inv_u, (float)si.y * inv_u);
        f.u[1] = bf16_pair((float)si.z / (0.01f * (float)P.rho0), (float)ncnt[i] / 32.f);
        f.u[2] = bf16_pair((float)wcnt[i] / 16.f, 0.f);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const bf16x8 w = frag_from_bf16(WnT + (size_t)(16 * t + r) * FPAD + 8 * g);
        const f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.v, w, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        const float bv = bn[16 * t + r];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float h = fmaxf(a[q] + bv, 0.f);
            H[(size_t)(m0 + 4 * g + q) * ldh + 16 * t + r] = h;
            Hs[wv][4 * g + q][16 * t + r] = (uint16_t)bf16_pair(h, 0.f);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bf16x8 h0 = frag_from_bf16(&Hs[wv][r][8 * g]), h1 = frag_from_bf16(&Hs[wv][r][32 + 8 * g]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        f32x4 p = f32x4{0.f, 0.f, 0.f, 0.f}, q = p;
        const uint16_t* wa = WaT + (size_t)(16 * t + r) * HID + 8 * g;
        const uint16_t* wb = WbT + (size_t)(16 * t + r) * HID + 8 * g;
        p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, frag_from_bf16(wa), p, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, frag_from_bf16(wb), q, 0, 0, 0);
        p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, frag_from_bf16(wa + 32), p, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, frag_from_bf16(wb + 32), q, 0, 0, 0);
        const float bv = bm[16 * t + r];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            Pm[(size_t)(m0 + 4 * g + k) * HID + 16 * t + r] = p[k] + bv;
            Qm[(size_t)(m0 + 4 * g + k) * HID + 16 * t + r] = q[k] + 0.f;
        }
    }
}

// Weights of one layer kernel (bf16 matrices transposed, 64 x K) and of what
// follows it: the next layer's P and Q, or (WaT null) the decoder.
struct LayerW {
    const uint16_t *WeT, *WcT, *WuT, *WaT, *WbT, *Wo1T;
    const float *be, *bu, *bm, *qn, *bo1, *Wo2, *bo2;  // qn: the next layer's wall vector
};

// What a training pass keeps of a layer: the sign bits of its messages (bit f
// of mask[e], e in CSR order), A in columns 64.. of X [N x 128] (whose first
// 64 columns are H), the update's pre-activation Z and the decoder's D1.
struct LayerKeep {
    const int32_t* eoff;
    unsigned long long* mask;
    float *X, *Z, *D1;
};

// One message-passing layer over the neighbour lists: for every node i, over
// its edges e (inner, then contact entries, in list order),
//   E0_e = relu(G_e We + be),  R_e = E0_e Wc,
//   m_e  = relu((P_i + (Q_j | qw)) + R_e),  A_i = sum_e m_e,
//   H_i <- H_i + relu([H_i | A_i] Wu + bu),
// then P, Q of the next layer (Q into the other buffer: this layer's is still
// gathered by other blocks) or the decoder's outputs Y.
//
// A block takes 4 NPW consecutive nodes, a wavefront NPW of them. Edge
// features are computed one edge per lane, 64 at a time, into LDS; the edge
// products run on the matrix cores in tiles of 16 edges, transposed
// (features as rows, edges as columns), and go through LDS to one lane per
// feature. There the message needs Q_j as one 256-byte row at an address that
// is uniform over the wavefront, and P_i stays in a register for a whole
// node; 16 row loads are in flight while the tile's products run. (Gathering
// P_i and Q_j in the matrix layout instead, with 16 bytes per lane, a row
// offset load per node and a stored 32-byte feature row per edge, took 597 us
// a layer and 398 us of features at 410k nodes and 8.1M edges.) The rows are
// read with buffer loads, whose row offset is one lane read: addresses and
// tests in the scalar unit cost as much issue time as the arithmetic
// (173 scalar instructions a tile, 553 us). The node
// update follows in the same block, on the rows it holds: wavefront w
// computes output columns 16 w .. 16 w + 15.
template <typename real, int NPW, bool TRAIN, bool BIG>
__global__ __launch_bounds__(256, 4) void k_gnn_layer(
    const KP<real>* __restrict__ Pt, const int32_t* __restrict__ tcase, int N, int lt,
    const uint32_t* __restrict__ nbr, const int32_t* __restrict__ ncnt, const uint32_t* __restrict__ wnb,
    const int32_t* __restrict__ wcnt, const R2<real>* __restrict__ geo, const R2<real>* __restrict__ wgeo,
    const R4<real>* __restrict__ st, LayerW W, const float* H, int ldh, float* Ho, int ldo, float* Pm,
    const float* __restrict__ Qm, float* __restrict__ Qn, float* __restrict__ Y, LayerKeep K)
{
    constexpr int NB = 4 * NPW;   // nodes per block
    constexpr int RT = NB / 16;   // row tiles of the node update
    static_assert(NB % 16 == 0 && TILE % NB == 0 && NPW < 64, "whole row tiles inside one case");
    __shared__ __align__(16) uint32_t Gs[4][64][4];
    __shared__ __align__(16) uint16_t Es[4][16][HID + 8];
    __shared__ __align__(16) float Ms[4][16][HID + 4];
    __shared__ __align__(16) uint16_t As[NB][HID + 8];
    __shared__ __align__(16) uint16_t Hb[NB][HID + 8];
    static_assert(sizeof(Ms) >= sizeof(float) * NB * (HID + 4), "the decoder's rows reuse Ms");
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int nb0 = blockIdx.x * NB;   // N is a multiple of TILE, so every node exists
    const int n0 = nb0 + wv * NPW;
    const KP<real>& P = Pt[tcase[nb0 / TILE]];
    if (W.WaT) special_rows(Qn, N, W.qn);
    const Rows<BIG> qrow(Qm, N + 2);
    const FeatScale fs = feat_scale(P);
    const int maxn = P.maxn, maxw = P.maxw;
    const real L0 = P.L[0], L1 = P.L[1];
    // lane p < NPW: inner count and (scanned) first edge of node n0 + p
    int nin = 0, tot = 0;
    if (lane < NPW && n0 + lane < P.fbase + P.nf) {
        nin = ncnt[n0 + lane];
        tot = nin + wcnt[n0 + lane];
    }
    int off = tot;
#pragma unroll
    for (int o = 1; o < NPW; o <<= 1) {
        const int a = __shfl_up(off, o);
        if (lane >= o) off += a;
    }
    const int ne = __builtin_amdgcn_readlane(off, NPW - 1);
    off -= tot;
    // weight fragments and the encoder bias of this lane, kept for all tiles
    bf16x8 wef[4], wcf[2][4];
    float bev[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        wef[t] = frag_from_bf16(W.WeT + (size_t)(16 * t + r) * FPAD + 8 * g);
#pragma unroll
        for (int k = 0; k < 2; ++k) wcf[k][t] = frag_from_bf16(W.WcT + (size_t)(16 * t + r) * HID + 32 * k + 8 * g);
#pragma unroll
        for (int q = 0; q < 4; ++q) bev[t][q] = W.be[16 * t + 4 * g + q];
    }
    const int ebase = TRAIN ? K.eoff[n0] : 0;
    // the reduction: lane = feature, running node `cur` (uniform)
    int cur = 0;
    float sum = 0.f;
    float pcur = Pm[(size_t)n0 * HID + lane];
    float pnext = Pm[(size_t)(n0 + (NPW > 1 ? 1 : 0)) * HID + lane];
    auto flush = [&]() __attribute__((always_inline)) {
        As[wv * NPW + cur][lane] = (uint16_t)bf16_pair(sum, 0.f);
        if constexpr (TRAIN) K.X[(size_t)(n0 + cur) * 2 * HID + HID + lane] = sum;
        sum = 0.f;
        ++cur;
        pcur = pnext;
        pnext = Pm[(size_t)(n0 + min(cur + 1, NPW - 1)) * HID + lane];
    };
    for (int eb = 0; eb < ne; eb += 64) {
        const int e = eb + lane;
        int dst = N + 1;
        int p = 0;
        unsigned long long starts;  // edges that are the first of a node after `cur`
        uint4 gq = make_uint4(0u, 0u, 0u, 0u);
        {
            int first = 0;
#pragma unroll
            for (int q = 1; q < NPW; ++q) {
                const int o = __builtin_amdgcn_readlane(off, q);
                if (e >= o) {
                    p = q;
                    first = o;
                }
            }
            const int i = n0 + p, ni = __shfl(nin, p);
            starts = __ballot(e == first && e < ne);
            if (e < ne) {
                const R2<real> oi = geo[i];
                const R4<real> si = st[i];
                const float devi = (float)si.z, vix = (float)si.x, viy = (float)si.y;
                const int k = e - first;
                const bool wall = k >= ni;
                const unsigned kk = (unsigned)(wall ? k - ni : k);
                const unsigned mx = (unsigned)(wall ? maxw : maxn), ui = (unsigned)i;
                const unsigned T1 = (1u << lt) - 1u;
                const size_t at = ((size_t)(ui >> (6 - lt)) * (mx >> lt) + (kk >> lt)) * 64 +
                                  (((ui & (63u >> lt)) << lt) | (kk & T1));
                const uint32_t ent = (wall ? wnb : nbr)[at];
                const int j = (int)(ent & NBR_MASK);
                const uint32_t code = ent >> NBR_SHIFT;
                const R2<real> oj = (wall ? wgeo : geo)[j];
                const float dx = (float)((oi.x - oj.x) - (real)((int)(code & 3u) - 1) * L0);
                const float dy = (float)((oi.y - oj.y) - (real)((int)((code >> 2) & 3u) - 1) * L1);
                float f[EFEAT];
                if (wall) {
                    edge_features(fs, dx, dy, -vix, -viy, 1.f, (fs.rho0 + devi) * (fs.gx * -dx + fs.gy * -dy), f);
                    dst = N;
                } else {
                    const R4<real> sj = st[j];
                    edge_features(fs, dx, dy, (float)sj.x - vix, (float)sj.y - viy, 0.f, fs.c2 * ((float)sj.z - devi), f);
                    dst = j;
                }
                gq = make_uint4(bf16_pair(f[0], f[1]), bf16_pair(f[2], f[3]), bf16_pair(f[4], f[5]),
                                bf16_pair(f[6], f[7]));
            }
        }
        dst = Rows<BIG>::key(dst);
        *(uint4*)&Gs[wv][lane][0] = gq;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int nt = min(4, (ne - eb + 15) >> 4);
        for (int t4 = 0; t4 < nt; ++t4) {
            // Q rows of the tile's edges
            float qv[16];
#pragma unroll
            for (int row = 0; row < 16; ++row)
                qv[row] = qrow.at(__builtin_amdgcn_readlane(dst, 16 * t4 + row), lane);
            // E0^T = We^T G^T: lane (r, g) holds edge r, features 16 t + 4 g + q
            Frag gf;
            gf.q = make_uint4(0u, 0u, 0u, 0u);
            if (g == 0) gf.q = *(const uint4*)&Gs[wv][16 * t4 + r][0];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wef[t], gf.v, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                uint2 pk;
                pk.x = bf16_pair(fmaxf(a[0] + bev[t][0], 0.f), fmaxf(a[1] + bev[t][1], 0.f));
                pk.y = bf16_pair(fmaxf(a[2] + bev[t][2], 0.f), fmaxf(a[3] + bev[t][3], 0.f));
                *(uint2*)&Es[wv][r][16 * t + 4 * g] = pk;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // R^T = Wc^T E0^T, two K steps of 32
            const bf16x8 e0 = frag_from_bf16(&Es[wv][r][8 * g]), e1 = frag_from_bf16(&Es[wv][r][32 + 8 * g]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wcf[0][t], e0, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wcf[1][t], e1, a, 0, 0, 0);
                *(float4*)&Ms[wv][r][16 * t + 4 * g] = make_float4(a[0], a[1], a[2], a[3]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // messages and per-node sums in list order (edgeless nodes too)
            float mrow[16];
#pragma unroll
            for (int row = 0; row < 16; ++row) mrow[row] = Ms[wv][row][lane];
            const unsigned heads = (unsigned)(starts >> (16 * t4)) & 0xffffu;
            unsigned long long sign = 0ull;  // lane row < 16: the sign bits of edge `row`
#pragma unroll
            for (int row = 0; row < 16; ++row) {
                if (heads & (1u << row)) {
                    const int to = __builtin_amdgcn_readlane(p, 16 * t4 + row);
                    while (cur < to) flush();
                }
                const float pre = (pcur + qv[row]) + mrow[row];
                if constexpr (TRAIN) {
                    const unsigned long long m = __ballot(pre > 0.f);
                    if (lane == row) sign = m;
                }
                sum += fmaxf(pre, 0.f);
            }
            if constexpr (TRAIN)
                if (lane < 16 && eb + 16 * t4 + lane < ne) K.mask[(size_t)(ebase + eb + 16 * t4 + lane)] = sign;
        }
    }
    while (cur < NPW) flush();
    __syncthreads();
    // node update, column tile wv
    const int col = 16 * wv + r;
    f32x4 acc[RT];
    float hold[RT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        const uint16_t* w = W.WuT + (size_t)col * 2 * HID + 8 * g;
        const float* h = H + (size_t)(nb0 + 16 * t + r) * ldh + 8 * g;
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_f32(h, true), frag_from_bf16(w), acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_f32(h + 32, true), frag_from_bf16(w + 32), acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_bf16(&As[16 * t + r][8 * g]), frag_from_bf16(w + 64), acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_bf16(&As[16 * t + r][32 + 8 * g]), frag_from_bf16(w + 96), acc[t], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) hold[t][q] = H[(size_t)(nb0 + 16 * t + 4 * g + q) * ldh + col];
    }
    __syncthreads();  // every wavefront has read the block's rows of H before they change
    const float bu = W.bu[col];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = 16 * t + 4 * g + q;
            const float z = acc[t][q] + bu;
            const float h = hold[t][q] + fmaxf(z, 0.f);
            if constexpr (TRAIN) K.Z[(size_t)(nb0 + row) * HID + col] = z;
            if (TRAIN || W.WaT) Ho[(size_t)(nb0 + row) * ldo + col] = h;  // (the decoder is the last reader)
            Hb[row][col] = (uint16_t)bf16_pair(h, 0.f);
        }
    __syncthreads();
    if (W.WaT) {
        const uint16_t *wa = W.WaT + (size_t)col * HID + 8 * g, *wb = W.WbT + (size_t)col * HID + 8 * g;
        const bf16x8 a0 = frag_from_bf16(wa), a1 = frag_from_bf16(wa + 32), b0 = frag_from_bf16(wb),
                     b1 = frag_from_bf16(wb + 32);
        const float bm = W.bm[col];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const bf16x8 h0 = frag_from_bf16(&Hb[16 * t + r][8 * g]), h1 = frag_from_bf16(&Hb[16 * t + r][32 + 8 * g]);
            f32x4 p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, a0, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            f32x4 q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, b0, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, a1, p, 0, 0, 0);
            q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1, b1, q, 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const size_t o = (size_t)(nb0 + 16 * t + 4 * g + k) * HID + col;
                Pm[o] = p[k] + bm;
                Qn[o] = q[k] + 0.f;
            }
        }
        return;
    }
    // decoder: D1 = relu(H Wo1 + bo1) through LDS, then the FP32 product with
    // Wo2, one thread per node and output (the same sums in the same order)
    float* D1 = &Ms[0][0][0];
    const uint16_t* wo = W.Wo1T + (size_t)col * HID + 8 * g;
    const float bo = W.bo1[col];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        f32x4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_bf16(&Hb[16 * t + r][8 * g]), frag_from_bf16(wo),
                                                          f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_bf16(&Hb[16 * t + r][32 + 8 * g]), frag_from_bf16(wo + 32), d, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float v = fmaxf(d[q] + bo, 0.f);
            D1[(16 * t + 4 * g + q) * (HID + 4) + col] = v;
            if constexpr (TRAIN) K.D1[(size_t)(nb0 + 16 * t + 4 * g + q) * HID + col] = v;
        }
    }
    __syncthreads();
    const int node = threadIdx.x / NOUT, c = threadIdx.x % NOUT;
    if (node >= NB) return;
    float y = W.bo2[c];
    for (int k = 0; k < HID; ++k) y += D1[node * (HID + 4) + k] * W.Wo2[k * NOUT + c];
    Y[(size_t)(nb0 + node) * NOUT + c] = y;
}

// ---------------------------------------------------------------------
// Backward of the edges. dM_e = dA_src(e) where message e was positive, else
// 0: it is formed from the sign bits and the source's row of dA wherever it
// is needed, so that no E x 64 array is stored (dM, R, E0, dE0 and the
// pre-activations were 256 bytes an edge each, written once and read up to
// four times). E0 is formed again from the edge features.

// A lane's value where its bit of the (uniform) word m is set, else 0.
__device__ __forceinline__ float where_bit(unsigned long long m, float v)
{
    return __builtin_amdgcn_inverse_ballot_w64(m) ? v : 0.f;
}

// Word k of a wavefront's 64 words.
__device__ __forceinline__ unsigned long long lane_word(unsigned long long v, int k)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, k), hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), k);
    return ((unsigned long long)hi << 32) | lo;
}

// Per node i (one wavefront, lane = feature): dP_i = sum_e dM_e,
// wsum_i = sum over wall edges of dM_e (for qw), and dQ_i = sum of dM over the
// inner edges that end at i, through the reverse of its own inner edges.
template <bool BIG>
__global__ __launch_bounds__(256) void k_gnn_node_bwd(int N, const int32_t* __restrict__ eoff,
                                                      const int32_t* __restrict__ edst,
                                                      const int32_t* __restrict__ erev,
                                                      const unsigned long long* __restrict__ mask,
                                                      const float* __restrict__ dA, float* __restrict__ dP,
                                                      float* __restrict__ dQ, float* __restrict__ wsum)
{
    const int i = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (i >= N) return;
    const int lane = threadIdx.x & 63;
    const Rows<BIG> rows(dA, N);
    const float da = dA[(size_t)i * HID + lane];
    const int e0 = eoff[i], e1 = eoff[i + 1];
    float sp = 0.f, sw = 0.f, sq = 0.f;
    for (int eb = e0; eb < e1; eb += 64) {
        unsigned long long own = 0ull, rev = 0ull;
        int at = 0, d = 0;
        if (eb + lane < e1) {
            const int e = eb + lane;
            own = mask[e];
            d = edst[e];
            const int rv = erev[e];
            if (d >= 0 && rv >= 0) {
                rev = mask[rv];
                at = Rows<BIG>::key(d);
            }
        }
        const unsigned long long wall = __ballot(d < 0);
        const int n = min(64, e1 - eb);
        for (int k = 0; k < n; k += 8) {  // (words past n are 0)
            float dj[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) dj[u] = rows.at(__builtin_amdgcn_readlane(at, k + u), lane);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float dm = where_bit(lane_word(own, k + u), da);
                sp += dm;
                if ((wall >> (k + u)) & 1ull) sw += dm;
                sq += where_bit(lane_word(rev, k + u), dj[u]);
            }
        }
    }
    dP[(size_t)i * HID + lane] = sp;
    dQ[(size_t)i * HID + lane] = sq;
    wsum[(size_t)i * HID + lane] = sw;
}

// Weight gradient of the edge product, dWc = E0^T dM over the edges [64 x 64]
// in row blocks, as k_wgrad: E0 and dM of a step's edges are formed in
// registers and staged transposed (E0 from the matrix cores with the edges as
// rows, so that a lane holds four consecutive edges of one feature; dM with
// one lane per feature, its row of dA under the edge's sign word).
template <bool BIG>
__global__ __launch_bounds__(256) void k_gnn_wgrad_edge(int E, int rows, int N, const float* __restrict__ G,
                                                        const int32_t* __restrict__ esrc,
                                                        const uint16_t* __restrict__ WeT, const float* __restrict__ be,
                                                        const unsigned long long* __restrict__ mask,
                                                        const float* __restrict__ dA, float* __restrict__ part)
{
    __shared__ __align__(16) uint16_t Xs[HID][WPAD];
    __shared__ __align__(16) uint16_t Zs[HID][WPAD];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const Rows<BIG> drow(dA, N);
    bf16x8 wef[4];
    float bev[4];
    f32x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        wef[t] = frag_from_bf16(WeT + (size_t)(16 * t + r) * FPAD + 8 * g);
        bev[t] = be[16 * t + r];
        acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int r0 = blockIdx.x * rows, r1 = min(r0 + rows, E);
    // this lane's edge of the wavefront's 16 (lanes r and r + 16 k alike)
    unsigned long long m = 0ull;
    int at = 0;
    bf16x8 gf;
    auto load = [&](int rb) __attribute__((always_inline)) {
        const int e = rb + 16 * w + r;
        const bool ok = e < r1;
        m = ok ? mask[e] : 0ull;
        at = ok ? esrc[e] : 0;
        gf = frag_from_f32(G + (size_t)(ok ? e : r0) * EFEAT, ok && g == 0);
    };
    load(r0);
    for (int rb = r0; rb < r1; rb += WROWS) {
        float z[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) z[q] = drow.at(__builtin_amdgcn_readlane(at, q), lane);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf, wef[t], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            *(uint2*)&Xs[16 * t + r][16 * w + 4 * g] =
                make_uint2(bf16_pair(fmaxf(a[0] + bev[t], 0.f), fmaxf(a[1] + bev[t], 0.f)),
                           bf16_pair(fmaxf(a[2] + bev[t], 0.f), fmaxf(a[3] + bev[t], 0.f)));
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) z[q] = where_bit(lane_word(m, q), z[q]);
        store_rows16(&Zs[lane][16 * w], z);
        __syncthreads();
        if (rb + WROWS < r1) load(rb + WROWS);
        wgrad_step<4>(Xs, Zs, w, r, g, acc);
        __syncthreads();
    }
    float* out = part + (size_t)blockIdx.x * HID * HID;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) out[(size_t)(16 * t + 4 * g + q) * HID + 16 * w + r] = acc[t][q];
}

// Backward of the edge encoder in row blocks: dE0 = sum over the layers (last
// first) of dM_l Wc_l^T, dZe = dE0 where E0 > 0, dWe = G^T dZe [FPAD x 64, the
// rows past the features 0] and dbe = column sums of dZe, row by row.
// Wavefront w computes feature columns 16 w .. 16 w + 15 of a step's 64 edges
// and keeps its six weight fragments in registers; the rows of dM_l, formed
// by the wavefront of their edges, go through LDS, one layer at a time.
struct EncBwd {
    const unsigned long long* mask[3];
    const float* dA[3];
    const uint16_t* WcN[3];
};
template <bool BIG>
__global__ __launch_bounds__(256) void k_gnn_enc_bwd(int E, int rows, int N, const float* __restrict__ G,
                                                     const int32_t* __restrict__ esrc,
                                                     const uint16_t* __restrict__ WeT, const float* __restrict__ be,
                                                     EncBwd B, float* __restrict__ part, float* __restrict__ bpart)
{
    __shared__ __align__(16) uint16_t Ds[WROWS][HID + 8];  // dM_l, edge rows
    __shared__ __align__(16) uint16_t Xs[16][WPAD];        // features (8 used), transposed
    __shared__ __align__(16) uint16_t Zs[HID][WPAD];       // dZe, transposed
    __shared__ float Zf[WROWS][HID];                       // dZe, FP32
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int col = 16 * w + r;
    const bf16x8 wef = frag_from_bf16(WeT + (size_t)col * FPAD + 8 * g);
    const float bev = be[col];
    bf16x8 wcf[3][2];
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int k = 0; k < 2; ++k) wcf[l][k] = frag_from_bf16(B.WcN[l] + (size_t)col * HID + 32 * k + 8 * g);
    for (int k = threadIdx.x; k < 16 * WPAD; k += 256) (&Xs[0][0])[k] = 0;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    const int r0 = blockIdx.x * rows, r1 = min(r0 + rows, E);
    __syncthreads();
    for (int rb = r0; rb < r1; rb += WROWS) {
        const int e = rb + 16 * w + r;
        const bool ok = e < r1;
        const int at = ok ? esrc[e] : 0;
        unsigned long long m[3];
#pragma unroll
        for (int l = 0; l < 3; ++l) m[l] = ok ? B.mask[l][e] : 0ull;
        // E0 of the step's edges: its sign, in the layout of the sums below
        uint32_t pos = 0;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int et = rb + 16 * t + r;
            const bf16x8 gf = frag_from_f32(G + (size_t)min(et, r1 - 1) * EFEAT, et < r1 && g == 0);
            if (t == w && g == 0) {  // this wavefront's edges: their features, transposed
                Frag f;
                f.v = gf;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    Xs[2 * k][16 * w + r] = (uint16_t)f.u[k];
                    Xs[2 * k + 1][16 * w + r] = (uint16_t)(f.u[k] >> 16);
                }
            }
            const f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf, wef, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) pos |= (a[q] + bev > 0.f ? 1u : 0u) << (4 * t + q);
        }
        f32x4 sum[4];
#pragma unroll
        for (int ll = 0; ll < 3; ++ll) {
            const int l = 2 - ll;
            const Rows<BIG> drow(B.dA[l], N);
            float z[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) z[q] = drow.at(__builtin_amdgcn_readlane(at, q), lane);
            if (ll) __syncthreads();  // the previous layer's rows have been read
#pragma unroll
            for (int q = 0; q < 16; ++q)
                Ds[16 * w + q][lane] = (uint16_t)bf16_pair(where_bit(lane_word(m[l], q), z[q]), 0.f);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_from_bf16(&Ds[16 * t + r][32 * k + 8 * g]), wcf[l][k],
                                                                a, 0, 0, 0);
                if (ll == 0) sum[t] = a;
                else sum[t] = sum[t] + a;
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = (pos >> (4 * t + q)) & 1u ? sum[t][q] : 0.f;
                Zf[16 * t + 4 * g + q][col] = v[q];
            }
            *(uint2*)&Zs[col][16 * t + 4 * g] = make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
        }
        __syncthreads();
        wgrad_step<1>(Xs, Zs, w, r, g, &acc);
        if (threadIdx.x < HID) {
            const int n = min(WROWS, r1 - rb);
#pragma unroll 16
            for (int q = 0; q < n; ++q) bsum += Zf[q][threadIdx.x];
        }
        __syncthreads();
    }
    float* out = part + (size_t)blockIdx.x * FPAD * HID;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        out[(size_t)(4 * g + q) * HID + col] = acc[q];
        out[(size_t)(16 + 4 * g + q) * HID + col] = 0.f;
    }
    if (threadIdx.x < HID) bpart[(size_t)blockIdx.x * HID + threadIdx.x] = bsum;
}

// out = src where mask > 0, else 0 (row strides given).
__global__ __launch_bounds__(256) void k_relu_mask(int M, const float* __restrict__ src, int lds,
                                                   const float* __restrict__ mask, int ldm, float* __restrict__ out,
                                                   int ldo)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)M * HID) return;
    const size_t r = idx / HID, c = idx % HID;
    out[r * ldo + c] = mask[r * ldm + c] > 0.f ? src[r * lds + c] : 0.f;
}

// dst[r][c] = src[r][c] for a [M x 64] block (row strides given).
__global__ __launch_bounds__(256) void k_copy64(int M, const float* __restrict__ src, int lds, float* __restrict__ dst,
                                                int ldd)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)M * HID) return;
    const size_t r = idx / HID, c = idx % HID;
    dst[r * ldd + c] = src[r * lds + c];
}

// Decoder output Y = D1 Wo2 + bo2 (FP32), one thread per node.
__global__ __launch_bounds__(256) void k_gnn_out(int N, const float* __restrict__ D1, const float* __restrict__ Wo2,
                                                 const float* __restrict__ bo2, float* __restrict__ Y)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    float y0 = bo2[0], y1 = bo2[1], y2 = bo2[2];
    const float* d = D1 + (size_t)i * HID;
    for (int k = 0; k < HID; ++k) {
        const float v = d[k];
        y0 += v * Wo2[k * NOUT + 0];
        y1 += v * Wo2[k * NOUT + 1];
        y2 += v * Wo2[k * NOUT + 2];
    }
    Y[(size_t)i * NOUT + 0] = y0;
    Y[(size_t)i * NOUT + 1] = y1;
    Y[(size_t)i * NOUT + 2] = y2;
}

// Loss: mean squared error over the fluid slots (count entries each of 3
// outputs): dY = 2 (Y - T) / (3 count); per-block partial sums of (Y - T)^2.
template <typename real>
__global__ __launch_bounds__(256) void k_gnn_loss(const KP<real>* __restrict__ Pt, const int32_t* __restrict__ tcase,
                                                  int ntiles, double inv_count, const float* __restrict__ Y,
                                                  const float* __restrict__ Tg, float* __restrict__ dY,
                                                  double* __restrict__ part)
{
    __shared__ double sh[4];
    const int tile = wave_tile();
    double s = 0.0;
    if (tile < ntiles) {
        const KP<real>& P = Pt[tcase[tile]];
        const int i = tile * TILE + (threadIdx.x & 63);
        const bool ok = i < P.fbase + P.nf;
        for (int c = 0; c < NOUT; ++c) {
            const float d = ok ? Y[(size_t)i * NOUT + c] - Tg[(size_t)i * NOUT + c] : 0.f;
            dY[(size_t)i * NOUT + c] = (float)(2.0 * (double)d * inv_count);
            s += (double)d * (double)d;
        }
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// Decoder backward: dZ1 = (dY Wo2^T) [D1 > 0] (one thread per node and
// feature) ...
__global__ __launch_bounds__(256) void k_gnn_out_bwd(int N, const float* __restrict__ D1, const float* __restrict__ dY,
                                                     const float* __restrict__ Wo2, float* __restrict__ dZ1)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)N * HID) return;
    const size_t i = idx / HID, k = idx % HID;
    const float* dy = dY + i * NOUT;
    const float v = dy[0] * Wo2[k * NOUT + 0] + dy[1] * Wo2[k * NOUT + 1] + dy[2] * Wo2[k * NOUT + 2];
    dZ1[idx] = D1[idx] > 0.f ? v : 0.f;
}

// ... and the partials of dWo2 = D1^T dY (64 x 3) and dbo2 = sum dY, per row
// block (195 values per block).
__global__ __launch_bounds__(256) void k_gnn_out_wgrad(int N, int rows, const float* __restrict__ D1,
                                                       const float* __restrict__ dY, float* __restrict__ part)
{
    const int t = threadIdx.x;
    if (t >= HID * NOUT + NOUT) return;
    const int r0 = blockIdx.x * rows, r1 = min(r0 + rows, N);
    float s = 0.f;
    if (t < HID * NOUT) {
        const int k = t / NOUT, c = t % NOUT;
        int r = r0;
        for (; r + 16 <= r1; r += 16) {  // 32 loads in flight
            float a[16], b[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                a[q] = D1[(size_t)(r + q) * HID + k];
                b[q] = dY[(size_t)(r + q) * NOUT + c];
            }
#pragma unroll
            for (int q = 0; q < 16; ++q) s += a[q] * b[q];
        }
        for (; r < r1; ++r) s += D1[(size_t)r * HID + k] * dY[(size_t)r * NOUT + c];
    } else {
        const int c = t - HID * NOUT;
        for (int r = r0; r < r1; ++r) s += dY[(size_t)r * NOUT + c];
    }
    part[(size_t)blockIdx.x * (HID * NOUT + NOUT) + t] = s;
}

// Adam (FP32 master parameters); c1 = 1/(1 - b1^t), c2 = 1/(1 - b2^t).
__global__ __launch_bounds__(256) void k_adam(int n, float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                              float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] = p[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// bf16 copies of one weight matrix W [K x 64] (FP32, row-major at src):
// transposed (64 x K, for products with W) and as is (K x 64, for products
// with W^T).
__global__ __launch_bounds__(256) void k_pack_w(int K, const float* __restrict__ W, uint16_t* __restrict__ WT,
                                                uint16_t* __restrict__ WN)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= K * HID) return;
    const int k = idx / HID, n = idx % HID;
    const uint16_t b = (uint16_t)bf16_bits(W[idx]);
    WT[(size_t)n * K + k] = b;
    WN[idx] = b;
}

// Surrogate state update over dt_c of every accepted case c:
// v' = v + a dt, x' = x + (v + v')/2 dt, rho' = rho + Drho dt; Drho becomes
// the density rate carried into the next half-step.
template <typename real>
__global__ __launch_bounds__(BLOCK) void k_gnn_apply(const KP<real>* __restrict__ Pt, const int32_t* __restrict__ tcase,
                                                     int ntiles, const double* __restrict__ dtc,
                                                     const int32_t* __restrict__ accept, const float* __restrict__ Y,
                                                     double* __restrict__ x0, double* __restrict__ x1,
                                                     R4<real>* __restrict__ st)
{
    const int tile = wave_tile();
    if (tile >= ntiles) return;
    const KP<real>& P = Pt[tcase[tile]];
    if (!accept[P.case_id]) return;
    const int i = tile * TILE + (threadIdx.x & 63);
    if (i >= P.fbase + P.nf) return;
    const double dt = dtc[P.case_id];
    const double gmag = sqrt((double)P.g[0] * P.g[0] + (double)P.g[1] * P.g[1] + (double)P.g[2] * P.g[2]);
    const double ax = (double)Y[(size_t)i * NOUT + 0] * gmag, ay = (double)Y[(size_t)i * NOUT + 1] * gmag;
    const double drho = (double)Y[(size_t)i * NOUT + 2] * 1e-3 * P.rho0d * P.u_ref / (0.5 * sqrt(P.rc2));
    R4<real> s = st[i];
    const double vx = (double)s.x, vy = (double)s.y;
    const double vx2 = vx + ax * dt, vy2 = vy + ay * dt;
    x0[i] = x0[i] + 0.5 * (vx + vx2) * dt;
    x1[i] = x1[i] + 0.5 * (vy + vy2) * dt;
    s.x = (real)vx2;
    s.y = (real)vy2;
    s.z = (real)((double)s.z + drho * dt);
    s.w = (real)drho;
    st[i] = s;
}

// Largest |rho/rho0 - 1| the surrogate would produce over dt_c, per case:
// per-tile maxima (k_diag_fin-style reduction on the host side of the call).
template <typename real>
__global__ __launch_bounds__(BLOCK) void k_gnn_check(const KP<real>* __restrict__ Pt, const int32_t* __restrict__ tcase,
                                                     int ntiles, const double* __restrict__ dtc,
                                                     const float* __restrict__ Y, const R4<real>* __restrict__ st,
                                                     double* __restrict__ tmax)
{
    const int tile = wave_tile();
    if (tile >= ntiles) return;
    const KP<real>& P = Pt[tcase[tile]];
    const int i = tile * TILE + (threadIdx.x & 63);
    double v = 0.0;
    if (i < P.fbase + P.nf) {
        const double drho = (double)Y[(size_t)i * NOUT + 2] * 1e-3 * P.rho0d * P.u_ref / (0.5 * sqrt(P.rc2));
        v = fabs(((double)st[i].z + drho * dtc[P.case_id]) / P.rho0d);
        if (v != v) v = 1e300;
    }
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) tmax[tile] = v;
}

// Targets of case c, given in original order (n x 3, FP64), into its slots.
template <typename real>
__global__ __launch_bounds__(BLOCK) void k_gnn_load_target(const KP<real>* __restrict__ Pt, int c,
                                                           const int32_t* __restrict__ id,
                                                           const double* __restrict__ src, float* __restrict__ Tg)
{
    const KP<real>& P = Pt[c];
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= P.nf) return;
    const int i = P.fbase + k;
    const int o = id[i];
    for (int q = 0; q < NOUT; ++q) Tg[(size_t)i * NOUT + q] = (float)src[(size_t)o * NOUT + q];
}

}  // namespace gnn
}  // namespace sphx
