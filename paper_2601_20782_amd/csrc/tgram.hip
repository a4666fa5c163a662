// Sample-space Gram matrix T = Obar Obar^T / n (Eq. eq:smat taken in sample
// space, Obar = O - mean over samples) from the factors of O, in FP64.
//
// For every network here a sample's O is a set of outer products: a dense
// layer l gives O_{W_l} = delta_l (x) a_{l-1} and O_{b_l} = delta_l; an RBM gives
// O_W = tanh(theta) (x) s, O_b = tanh(theta), O_a = s.  Writing each layer as a
// pair of per-sample factors U (rows) and V (columns), and c = 1 when V is
// also a block of O on its own (the RBM's visible bias), the dot product of
// two samples' O is
//     K_kl = sum_layers (U_k.U_l + c) (V_k.V_l + 1) - c,
// so K needs Gram matrices of the factors (contractions over a few thousand
// values) instead of one over all P parameters.  Centring is exact algebra:
//     T_kl = (K_kl - v_k - v_l + |mu|^2) / n,   v_k = O_k . mu,
// with mu = mean of O, which per layer is the matrix (1/n) [U,1]^T [V,1]
// (masked to the blocks that exist).  Means, v and K are FP64 throughout
// (products of FP32 factors are exact in FP64); T is rounded to FP32 once.
//
// The vector-Jacobian product O^T g is the same kind of sum, sum_k g_k [U_k,1] (x) [V_k,1] per layer, so it comes
// from the same kernel as the means.
//
// Kernels, all on the FP64 matrix cores (v_mfma_f64_16x16x4f64): fac_outer (one block per 64 x 64 tile of a layer's
// mean matrix and range of samples; the ranges summed in order by fac_mean_reduce or, into parameter order, by
// fac_vjp_reduce), fac_v (per-sample bilinear forms, partials per row tile summed in fixed order), fac_gram (one
// block per 64 x 64 tile of T's upper triangle).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "internal.h"

namespace nqs {

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct FacLayer {
    const float *U;   // [n][ldu], first du columns used
    const float *V;   // [n][ldv], first dv columns used; NULL: the spins S
    const int8_t *S;
    int64_t ldu, ldv;
    int du, dv;
    int c;            // 1: V is also a block of O by itself
    double *M;        // [(du + 1) x (dv + 1)] masked mean matrix (inside FacArgs::Mall)
    int64_t moff;     // offset of M in Mall
    int64_t mt0;      // first mean tile of this layer (flattened over layers)
    int64_t vs0;      // first v-partial slot of this layer
};

struct FacArgs {
    FacLayer lay[NQS_MAX_LAYERS + 1];
    int L;
    int64_t n;
    double *Mall;     // [mtot] the layers' mean matrices, one after the other
    double *mpart;    // [splits][mtot] per-split sums of the mean matrices
    int64_t mtot;
    int splits;       // sample ranges of the mean sums
    double *m2part;   // [m2blocks] sums of squares of Mall per reduction block
    int m2blocks;
    double *vpart;    // [slots][n]
    int64_t slots;
    double *v;        // [n]
    double *m2;       // [1]
    float *T;         // [n][n]
    int64_t nt;       // 64-row tiles per side of T
};

constexpr int kFT = 64;    // tile side
constexpr int kFK = 32;    // contraction steps staged per barrier by fac_outer and fac_v

__device__ inline int fac_layer_of(const FacArgs &A, int64_t t, bool vslots)
{
    int l = 0;
    while (l + 1 < A.L && t >= (vslots ? A.lay[l + 1].vs0 : A.lay[l + 1].mt0)) ++l;
    return l;
}

// value of the augmented factor [F, 1] at (row k, column j), zero outside
__device__ inline double fac_aug(const float *F, int64_t ld, int d, int64_t n, int64_t k, int64_t j)
{
    if (k >= n || j > d) return 0.0;
    return j == d ? 1.0 : (double)F[k * ld + j];
}

// The vector-Jacobian product's parameter order: with c = 1 (RBM) [row du, column dv, inner block], else [inner block,
// column dv] of each layer in turn.  The first parameter of layer l, and the place in it of entry (r, c) of its sums
// (-1: no parameter).
__device__ __forceinline__ int64_t fac_vjp_first(const FacArgs &A, int l)
{
    int64_t off = 0;
    for (int i = 0; i < l; ++i) off += (int64_t)A.lay[i].du * (A.lay[i].dv + 1) + (A.lay[i].c ? A.lay[i].dv : 0);
    return off;
}
__device__ __forceinline__ int64_t fac_vjp_place(const FacLayer &y, int r, int c)
{
    if (r < y.du) return c < y.dv ? (y.c ? y.dv + y.du : 0) + (int64_t)r * y.dv + c : (y.c ? y.dv : (int64_t)y.du * y.dv) + r;
    return c < y.dv && y.c ? c : -1;
}

// Sums of g_k [U_k,1] (x) [V_k,1] (g = 1 without `g`) over the samples of one split (blockIdx.y), one 64 x 64 tile
// of one layer per block (blockIdx.x), to mpart, or added to it (`add`), or, where one split holds all samples, straight
// to the gradient `vjp` (400 x 1600 RBM, 100 samples: 252 us with the sums written, read and reduced, 196 us without).
// The products of two FP32 factors and of g with one are exact in FP64.  Both operands are read along the samples, 32 of
// them per barrier with the next 32 already in registers (the row stride of 80 floats spreads a fragment read over all
// banks): a block's four waves then wait for the matrix cores, 2048 cycles per 32 samples, and not for memory.  Mean
// matrices of the 100-400-200 network, 6000 samples: 118 us on the vector units, 90 us (1.45 GFLOP; 64-bit vector and
// matrix rates are alike, the vector form waited for its LDS reads).
constexpr int kOutLd = 80;
__global__ void __launch_bounds__(256) fac_outer_kernel(FacArgs A, const float *__restrict__ g, int add,
                                                        float *__restrict__ vjp)
{
    __shared__ float Us[2][kFK * kOutLd], Vs[2][kFK * kOutLd], gs[2][kFK];
    const int l = fac_layer_of(A, blockIdx.x, false);
    const FacLayer &y = A.lay[l];
    const int64_t t = blockIdx.x - y.mt0;
    const int ctiles = (y.dv + 1 + kFT - 1) / kFT;
    const int r0 = (int)(t / ctiles) * kFT, c0 = (int)(t % ctiles) * kFT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, la = lane & 15, lk = lane >> 4;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int64_t kb = blockIdx.y * A.n / A.splits, ke = (blockIdx.y + 1) * A.n / A.splits;
    const int j = lane, s0 = wave;   // staging: column j of the samples s0, s0 + 4, ...
    float uv[kFK / 4], vv[kFK / 4], gv = 0.0f;
    // every load is made, from a valid place; columns past the last feed sums that are not stored
    const int r = r0 + j, c = c0 + j, rc = min(r, y.du - 1), cc = min(c, y.dv - 1);
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int i = 0; i < kFK / 4; ++i) {
            const int64_t k = k0 + s0 + 4 * i, kc = min(k, A.n - 1);
            const float u = y.U[kc * y.ldu + rc], v = y.V ? y.V[kc * y.ldv + cc] : (float)y.S[kc * y.ldv + cc];
            uv[i] = k >= ke ? 0.0f : r == y.du ? 1.0f : u;
            vv[i] = k >= ke ? 0.0f : c == y.dv ? 1.0f : v;
        }
        if (tid < kFK) gv = k0 + tid >= ke ? 0.0f : g ? g[k0 + tid] : 1.0f;
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kFK / 4; ++i) {
            Us[buf][(s0 + 4 * i) * kOutLd + j] = uv[i];
            Vs[buf][(s0 + 4 * i) * kOutLd + j] = vv[i];
        }
        if (tid < kFK) gs[buf][tid] = gv;
    };
    f64x4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    load(kb);
    store(0);
    int buf = 0;
    for (int64_t k0 = kb; k0 < ke; k0 += kFK) {
        __syncthreads();
        const bool more = k0 + kFK < ke;
        if (more) load(k0 + kFK);
#pragma unroll
        for (int s = 0; s < kFK / 4; ++s) {
            const int kk = 4 * s + lk;
            const double w = (double)gs[buf][kk];
            double u[2], v[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u[q] = w * (double)Us[buf][kk * kOutLd + wm + 16 * q + la];
                v[q] = (double)Vs[buf][kk * kOutLd + wn + 16 * q + la];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[a], v[b], acc[a][b], 0, 0, 0);
        }
        if (more) store(buf ^ 1);
        buf ^= 1;
    }
    // D[i][j] of a 16 x 16 FP64 block: j = lane % 16, i = lane / 16 + 4 * register
    double *out = A.mpart + (int64_t)blockIdx.y * A.mtot + y.moff;
    if (vjp) vjp += fac_vjp_first(A, l);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + wm + 16 * a + lk + 4 * q, c = c0 + wn + 16 * b + la;
                if (r > y.du || c > y.dv) continue;
                if (vjp) {
                    const int64_t p = fac_vjp_place(y, r, c);
                    if (p >= 0) vjp[p] = (float)(0.0 + acc[a][b][q]);
                    continue;
                }
                double *o = out + (int64_t)r * (y.dv + 1) + c;
                *o = add ? *o + acc[a][b][q] : acc[a][b][q];
            }
}

// Entry e of the layers' sums, the splits added in order (eight loads in flight).
__device__ __forceinline__ double fac_split_sum(const FacArgs &A, int64_t e)
{
    double s = 0.0;
#pragma unroll 8
    for (int sp = 0; sp < A.splits; ++sp) s += A.mpart[(int64_t)sp * A.mtot + e];
    return s;
}

// The sums of fac_outer_kernel as the gradient in parameter order
__global__ void __launch_bounds__(256) fac_vjp_reduce_kernel(FacArgs A, float *__restrict__ out)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= A.mtot) return;
    int l = 0;
    while (l + 1 < A.L && e >= A.lay[l + 1].moff) ++l;
    const FacLayer &y = A.lay[l];
    const int64_t q = e - y.moff;
    const int r = (int)(q / (y.dv + 1)), c = (int)(q - (int64_t)r * (y.dv + 1));
    const int64_t p = fac_vjp_place(y, r, c);
    if (p >= 0) out[fac_vjp_first(A, l) + p] = (float)fac_split_sum(A, e);
}

// M_l = (1/n) (sum of the splits in order), masked: the (du, dv) corner is 0 and
// row du (the mean of V alone) is kept only when c = 1.  Per block, the sum of
// squares of its entries goes to m2part.
__global__ void __launch_bounds__(256) fac_mean_reduce_kernel(FacArgs A)
{
    __shared__ double red[256];
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    double m = 0.0;
    if (e < A.mtot) {
        int l = 0;
        while (l + 1 < A.L && e >= A.lay[l + 1].moff) ++l;
        const FacLayer &y = A.lay[l];
        const int64_t q = e - y.moff;
        const int r = (int)(q / (y.dv + 1)), c = (int)(q - (int64_t)r * (y.dv + 1));
        m = fac_split_sum(A, e) / (double)A.n;
        if (r == y.du && (c == y.dv || !y.c)) m = 0.0;
        A.Mall[e] = m;
    }
    red[threadIdx.x] = m * m;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) A.m2part[blockIdx.x] = red[0];
}

// vpart[slot][k] = sum over the slot's 64 rows r of [U_k,1]_r (M [V_k,1])_r: a 64 samples x 64 rows tile of
// [V,1] M^T on the FP64 matrix cores, then the products with [U,1] summed over the rows.  32 columns per barrier,
// the next ones in registers meanwhile; row strides of 36 words (of either size) spread a fragment read over the
// banks.  100-400-200, 6000 samples: 157 us on the vector units (eight LDS reads per 16 multiply-adds), 74 us.
constexpr int kVLd = 36;
__global__ void __launch_bounds__(256) fac_v_kernel(FacArgs A)
{
    __shared__ float Vs[kFT * kVLd];
    __shared__ double Ms[kFT * kVLd];
    __shared__ double part[2][kFT];
    const int l = fac_layer_of(A, blockIdx.y, true);
    const FacLayer &y = A.lay[l];
    const int r0 = (int)(blockIdx.y - y.vs0) * kFT;
    const int64_t k0 = (int64_t)blockIdx.x * kFT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, la = lane & 15, lk = lane >> 4;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int ldm = y.dv + 1;
    const int sc = tid & 31, sr = tid >> 5;   // staging: column sc of the rows sr, sr + 8, ...
    float vv[8];
    double mv[8];
    auto load = [&](int c0) {
        const int c = c0 + sc;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t k = k0 + sr + 8 * i;
            const int r = r0 + sr + 8 * i;
            const float v = y.V[min(k, A.n - 1) * y.ldv + min(c, y.dv - 1)];
            const double m = y.M[(int64_t)min(r, y.du) * ldm + min(c, y.dv)];
            vv[i] = c > y.dv ? 0.0f : c == y.dv ? 1.0f : v;
            mv[i] = c > y.dv ? 0.0 : m;
        }
    };
    f64x4 acc[2][2];   // [sample block][row block]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    load(0);
    for (int c0 = 0; c0 <= y.dv; c0 += kFK) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            Vs[(sr + 8 * i) * kVLd + sc] = vv[i];
            Ms[(sr + 8 * i) * kVLd + sc] = mv[i];
        }
        __syncthreads();
        if (c0 + kFK <= y.dv) load(c0 + kFK);
#pragma unroll
        for (int s = 0; s < kFK / 4; ++s) {
            double v[2], m[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                v[q] = (double)Vs[(wm + 16 * q + la) * kVLd + 4 * s + lk];
                m[q] = Ms[(wn + 16 * q + la) * kVLd + 4 * s + lk];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[a], m[b], acc[a][b], 0, 0, 0);
        }
    }
    // D[i][j]: j = lane % 16 (row), i = lane / 16 + 4 * register (sample); the 16 lanes of a sample in a fixed
    // order, then the two waves that share its samples
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = wm + 16 * a + lk + 4 * q;
            double s = 0.0;
#pragma unroll
            for (int b = 0; b < 2; ++b)
                s = fma(fac_aug(y.U, y.ldu, y.du, A.n, k0 + i, r0 + wn + 16 * b + la), acc[a][b][q], s);
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) s += __shfl_xor(s, o, 16);
            if (la == 0) part[wave & 1][i] = s;
        }
    __syncthreads();
    if (tid < kFT && k0 + tid < A.n) A.vpart[(int64_t)blockIdx.y * A.n + k0 + tid] = part[0][tid] + part[1][tid];
}

// v[k] = sum of the slots in order; block 0 also sums |mu|^2 from the reduction blocks
__global__ void __launch_bounds__(256) fac_vsum_kernel(FacArgs A)
{
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k < A.n) {
        double s = 0.0;
        for (int64_t q = 0; q < A.slots; ++q) s += A.vpart[q * A.n + k];
        A.v[k] = s;
    }
    if (blockIdx.x != 0) return;
    __shared__ double red[256];
    double s = 0.0;
    for (int b = threadIdx.x; b < A.m2blocks; b += blockDim.x) s += A.m2part[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) A.m2[0] = red[0];
}

// Tile (bi, bj), bi <= bj, of the upper triangle in row-major order.
__device__ inline void fac_tile(int64_t t, int64_t nt, int64_t &bi, int64_t &bj)
{
    const double a = (double)(2 * nt + 1);
    int64_t r = (int64_t)((a - sqrt(a * a - 8.0 * (double)t)) * 0.5);
    r = r < 0 ? 0 : (r > nt - 1 ? nt - 1 : r);
    auto start = [nt](int64_t row) { return row * nt - row * (row - 1) / 2; };
    while (r > 0 && start(r) > t) --r;
    while (r + 1 < nt && start(r + 1) <= t) ++r;
    bi = r;
    bj = r + (t - start(r));
}

constexpr int kGThreads = 512;
constexpr int kGStep = 32;   // contraction steps per barrier of the matrix-core kernel
constexpr int kGLd = 36;     // LDS row stride (floats): a fragment read covers all banks once

// acc[b] (two 16 x 16 blocks, the wave's 16 x 32 part of the tile) += F_I F_J^T over the first d columns.  The next 32
// columns are loaded into registers during the products of the current ones and stored into the other LDS buffer,
// one barrier per step: 1024 cycles of products a wave against one memory latency.
__device__ __forceinline__ void fac_gram_accumulate(const float *__restrict__ F, int64_t ld, int d, int64_t n,
                                                    int64_t I0, int64_t J0, float *As, float *Bs, f64x4 (&acc)[2])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 16, wn = (wave & 1) * 32;
    const int sc = tid & 31, sr = tid >> 5;   // staging: column sc of the rows sr, sr + 16, ...
    const int li = lane & 15, lk = lane >> 4;
    float av[4], bv[4];
    auto load = [&](int k0) {
        // every load is made, from a valid place (a branch around a load waits for all loads in flight); rows past
        // the last feed outputs that are not stored
        const int k = k0 + sc, kc = min(k, d - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t gi = min(I0 + sr + 16 * i, n - 1), gj = min(J0 + sr + 16 * i, n - 1);
            const float a = F[gi * ld + kc], b = F[gj * ld + kc];
            av[i] = k < d ? a : 0.0f;
            bv[i] = k < d ? b : 0.0f;
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            As[(buf * kFT + sr + 16 * i) * kGLd + sc] = av[i];
            Bs[(buf * kFT + sr + 16 * i) * kGLd + sc] = bv[i];
        }
    };
    load(0);
    __syncthreads();   // the previous contraction's last reads
    store(0);
    int buf = 0;
    for (int k0 = 0; k0 < d; k0 += kGStep) {
        __syncthreads();
        const bool more = k0 + kGStep < d;
        if (more) load(k0 + kGStep);
        const float *Ab = As + buf * kFT * kGLd, *Bb = Bs + buf * kFT * kGLd;
#pragma unroll
        for (int s = 0; s < kGStep / 4; ++s) {
            const int kk = s * 4 + lk;
            const double a = (double)Ab[(wm + li) * kGLd + kk];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)Bb[(wn + 16 * j + li) * kGLd + kk], acc[j], 0,
                                                              0, 0);
        }
        if (more) store(buf ^ 1);
        buf ^= 1;
    }
}

// Bound by the FP64 matrix cores (busy in 67 % of the cycles).  Eight waves of 16 x 32 hold K and two products in 48
// registers each, so that two blocks (four waves per SIMD) share a CU.  T of 6000 samples of the 100-400-200 network:
// 1328 us with four waves of 32 x 32 and loads between two barriers of 16 columns, 1288 with the loads ahead at one
// wave per SIMD, 946 at two, 923-938 (43 TFLOP/s on the computed tiles) now; 10 x 10 RBM, 4096 samples 202 -> 158 us.
__global__ void __launch_bounds__(kGThreads, 4) fac_gram_kernel(FacArgs A)
{
    __shared__ float As[2 * kFT * kGLd], Bs[2 * kFT * kGLd];
    // consecutive tiles (which share their row panel) on one XCD
    const int64_t tiles = A.nt * (A.nt + 1) / 2;
    const int64_t x = blockIdx.x, g = gridDim.x;
    const int64_t q8 = g >> 3, r8 = g & 7, xcd = x & 7;
    const int64_t t = xcd * q8 + min(xcd, r8) + (x >> 3);
    if (t >= tiles) return;
    int64_t bi, bj;
    fac_tile(t, A.nt, bi, bj);
    const int64_t I0 = bi * kFT, J0 = bj * kFT;

    f64x4 K[2], gu[2], gv[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) K[b] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int l = 0; l < A.L; ++l) {
        const FacLayer &y = A.lay[l];
#pragma unroll
        for (int b = 0; b < 2; ++b) gu[b] = gv[b] = f64x4{0.0, 0.0, 0.0, 0.0};
        fac_gram_accumulate(y.U, y.ldu, y.du, A.n, I0, J0, As, Bs, gu);
        fac_gram_accumulate(y.V, y.ldv, y.dv, A.n, I0, J0, As, Bs, gv);
        const double c = (double)y.c;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) K[b][r] += fma(gu[b][r] + c, gv[b][r] + 1.0, -c);
    }

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 16, wn = (wave & 1) * 32;
    const double inv = 1.0 / (double)A.n, m2 = A.m2[0];
    // D[i][j] of a 16 x 16 FP64 block: j = lane % 16, i = lane / 16 + 4 * register
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t gi = I0 + wm + (lane >> 4) + 4 * r;
            const int64_t gj = J0 + wn + 16 * b + (lane & 15);
            if (gi >= A.n || gj >= A.n || (bi == bj && gi > gj)) continue;
            const float tv = (float)((K[b][r] - A.v[gi] - A.v[gj] + m2) * inv);
            A.T[gi * A.n + gj] = tv;
            if (gi != gj) A.T[gj * A.n + gi] = tv;
        }
}

__global__ void spins_to_f32_kernel(const int8_t *__restrict__ s, int64_t count, float *__restrict__ out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < count) out[i] = (float)s[i];
}

// ---- host ----

// Launch geometry shared by the workspace size and the launch.
struct FacPlan {
    int64_t mt = 0, mtot = 0, vs = 0;
    int splits = 1, m2blocks = 1;
};

static FacPlan fac_plan(const FacLayerDesc *lay, int L, int64_t n)
{
    FacPlan p;
    for (int l = 0; l < L; ++l) {
        const int64_t rt = (lay[l].du + 1 + kFT - 1) / kFT, ct = (lay[l].dv + 1 + kFT - 1) / kFT;
        p.mt += rt * ct;
        p.mtot += (int64_t)(lay[l].du + 1) * (lay[l].dv + 1);
        p.vs += rt;
    }
    // sample splits for about two blocks per compute unit, at least 64 samples each (more splits only cost their sum:
    // 10 x 10 RBM, 4096 samples: 64 splits 27 us and 19 us for their sum, 32 splits 18 us and 6 us)
    const int64_t want = ((int64_t)device_cus() * 2 + p.mt - 1) / p.mt;
    p.splits = (int)std::max<int64_t>(1, std::min<int64_t>({want, n / 64, 1024}));
    p.m2blocks = (int)((p.mtot + 255) / 256);
    return p;
}

static size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t fac_workspace_bytes(const FacLayerDesc *lay, int L, int64_t n)
{
    const FacPlan p = fac_plan(lay, L, n);
    return round256(sizeof(double) * (size_t)p.mtot) + round256(sizeof(double) * (size_t)p.splits * p.mtot) +
           round256(sizeof(double) * (size_t)p.m2blocks) + round256(sizeof(double) * (size_t)p.vs * (size_t)n) +
           round256(sizeof(double) * (size_t)n) + 256;
}

// the layers and their places in the mean matrices and slots
static FacArgs fac_args(const FacLayerDesc *lay, int L, int64_t n, const FacPlan &p, double *Mall)
{
    FacArgs A{};
    A.L = L;
    A.n = n;
    A.mtot = p.mtot;
    A.splits = p.splits;
    A.m2blocks = p.m2blocks;
    A.slots = p.vs;
    A.Mall = Mall;
    int64_t mt = 0, vs = 0, moff = 0;
    for (int l = 0; l < L; ++l) {
        FacLayer &y = A.lay[l];
        y.U = lay[l].U;
        y.V = lay[l].V;
        y.S = lay[l].S;
        y.ldu = lay[l].ldu;
        y.ldv = lay[l].ldv;
        y.du = lay[l].du;
        y.dv = lay[l].dv;
        y.c = lay[l].c;
        y.moff = moff;
        y.M = Mall + moff;
        moff += (int64_t)(y.du + 1) * (y.dv + 1);
        y.mt0 = mt;
        mt += (int64_t)((y.du + 1 + kFT - 1) / kFT) * ((y.dv + 1 + kFT - 1) / kFT);
        y.vs0 = vs;
        vs += (y.du + 1 + kFT - 1) / kFT;
    }
    return A;
}

size_t fac_vjp_bytes(const FacLayerDesc *lay, int L, int64_t n)
{
    const FacPlan p = fac_plan(lay, L, n);
    return round256(sizeof(double) * (size_t)p.splits * p.mtot);
}

nqs_status launch_fac_vjp(const FacLayerDesc *lay, int L, int64_t n, int64_t n_first, const float *g, bool add,
                          float *vjp_out, void *wsp, hipStream_t stream)
{
    if (L < 1 || L > NQS_MAX_LAYERS + 1) return set_error(NQS_EINVAL, "bad factor layer count");
    const FacPlan p = fac_plan(lay, L, n_first);   // every chunk fills the first one's splits
    FacArgs A = fac_args(lay, L, n, p, nullptr);
    A.mpart = (double *)wsp;
    if (p.mt > INT32_MAX || (p.mtot + 255) / 256 > INT32_MAX) return set_error(NQS_EINVAL, "network too large");
    const bool whole = vjp_out && !add && p.splits == 1;
    hipLaunchKernelGGL(fac_outer_kernel, dim3((unsigned)p.mt, (unsigned)p.splits), dim3(256), 0, stream, A, g, add ? 1 : 0,
                       whole ? vjp_out : nullptr);
    if (vjp_out && !whole)
        hipLaunchKernelGGL(fac_vjp_reduce_kernel, dim3((unsigned)((p.mtot + 255) / 256)), dim3(256), 0, stream, A,
                           vjp_out);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

nqs_status launch_fac_gram(const FacLayerDesc *lay, int L, int64_t n, float *T, void *wsp, hipStream_t stream)
{
    if (L < 1 || L > NQS_MAX_LAYERS + 1) return set_error(NQS_EINVAL, "bad factor layer count");
    const FacPlan p = fac_plan(lay, L, n);
    FacArgs A = fac_args(lay, L, n, p, (double *)wsp);
    A.T = T;
    char *ws = (char *)wsp;
    ws += round256(sizeof(double) * (size_t)p.mtot);
    A.mpart = (double *)ws;
    ws += round256(sizeof(double) * (size_t)p.splits * p.mtot);
    A.m2part = (double *)ws;
    ws += round256(sizeof(double) * (size_t)p.m2blocks);
    A.vpart = (double *)ws;
    ws += round256(sizeof(double) * (size_t)p.vs * (size_t)n);
    A.v = (double *)ws;
    ws += round256(sizeof(double) * (size_t)n);
    A.m2 = (double *)ws;
    A.nt = (n + kFT - 1) / kFT;
    const int64_t tiles = A.nt * (A.nt + 1) / 2;
    const int64_t ktiles = (n + kFT - 1) / kFT;
    if (tiles > INT32_MAX || p.mt > INT32_MAX || ktiles > INT32_MAX || p.vs > 65535 || p.m2blocks > INT32_MAX / 2)
        return set_error(NQS_EINVAL, "sample-space Gram matrix too large");

    hipLaunchKernelGGL(fac_outer_kernel, dim3((unsigned)p.mt, (unsigned)p.splits), dim3(256), 0, stream, A,
                       (const float *)nullptr, 0, (float *)nullptr);
    hipLaunchKernelGGL(fac_mean_reduce_kernel, dim3((unsigned)p.m2blocks), dim3(256), 0, stream, A);
    hipLaunchKernelGGL(fac_v_kernel, dim3((unsigned)ktiles, (unsigned)p.vs), dim3(256), 0, stream, A);
    hipLaunchKernelGGL(fac_vsum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, A);
    hipLaunchKernelGGL(fac_gram_kernel, dim3((unsigned)tiles), dim3(kGThreads), 0, stream, A);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

void launch_spins_to_f32(const int8_t *s, int64_t count, float *out, hipStream_t stream)
{
    hipLaunchKernelGGL(spins_to_f32_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, s, count,
                       out);
}

}  // namespace nqs
