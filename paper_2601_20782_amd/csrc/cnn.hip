// Residual convolutional network (App. H) on an L x L periodic lattice:
//   h0 = Conv(s);  h <- h + Conv(phi(Conv(phi(LN(h)))))  (R blocks);
//   log psi = sum over sites and channels of LN(h).
// Conv: 3 x 3 cross-correlation with circular padding and a bias per output
// channel; LN: per site over the F channels, learnable scale and shift,
// epsilon 1e-6; phi: GELU, tanh form.  Reduced precision: the parameters are
// rounded to the sampling format, and so is the input of every convolution
// after the first; sums, LN, GELU and the residual stream are FP32.
//
// Two forms.  With 16 or 32 channels the sampler and the local energies evaluate
// batches of configurations, convolutions on the matrix cores (second half of
// this file).  The other networks, log psi and the log-derivatives take one
// configuration per workgroup, activations in LDS ([site][channel], FP32),
// weights read from the copy ([in channel][offset][out channel], so consecutive
// threads (out channels) read consecutive words): the sampler one chain per
// workgroup (proposal, forward pass, decision), the local energy one sample per
// workgroup (the sample and its N flips).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "common.h"
#include "internal.h"

namespace nqs {

constexpr int kCnnThreads = 256;
constexpr float kLnEps = 1e-6f;

int64_t cnn_num_params(int F, int R)
{
    return 10 * (int64_t)F + (int64_t)R * (2 * F + 2 * (9 * (int64_t)F * F + F)) + 2 * (int64_t)F;
}

// ---- copy: round the FP64 master, rearrange each convolution's weights ----

struct CnnSeg {
    int64_t start, len;
    int conv;   // 0: copied as is; else a convolution with `conv` input channels: [o][c][k] -> [c][k][o]
    int F;
};

__global__ void cnn_build_kernel(const double *__restrict__ master, int64_t P, int dtype, const CnnSeg *__restrict__ segs,
                                 int nseg, float *__restrict__ out)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= P) return;
    int s = 0;
    while (s + 1 < nseg && q >= segs[s + 1].start) ++s;
    const CnnSeg g = segs[s];
    const float v = (float)round_to_dtype(master[q], dtype);
    const int64_t r = q - g.start;
    if (g.conv == 0) {
        out[q] = v;
    } else {
        const int C = g.conv, F = g.F;
        const int64_t o = r / (9 * C), rem = r - o * 9 * C, c = rem / 9, k = rem - c * 9;
        out[g.start + (c * 9 + k) * F + o] = v;
    }
}

// Operands of the matrix-core convolutions from the rearranged FP32 values ([in][offset][out]):
// wmf, FP32, [offset][out][(in % 4) F / 4 + in / 4] (F a multiple of 4; a lane of the 4-deep
// product reads its channels as consecutive words), and for the 16-bit copies wmc, codes,
// [offset][out][in]; the values are exact in the copy's format.
__global__ void cnn_build_mc_kernel(CnnDev n, int64_t total)
{
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= total) return;
    const int F = n.F;
    const int64_t per = 9 * (int64_t)F * F;
    const int rj = (int)(q / per);
    const int64_t e = q - rj * per;
    const int k = (int)(e / ((int64_t)F * F)), o = (int)((e / F) % F), c = (int)(e % F);
    const int r = rj >> 1;
    const float *W = n.p + ((rj & 1) ? n.w2[r] : n.w1[r]);
    const float v = W[((int64_t)c * 9 + k) * F + o];
    if (F % 4 == 0) n.wmf[q - c + (c % 4) * (F / 4) + c / 4] = v;
    if (n.dtype == kF32) return;
    if (n.dtype == kBF16) {
        reinterpret_cast<uint16_t *>(n.wmc)[q] = (uint16_t)(__float_as_uint(v) >> 16);
    } else {
        const _Float16 hv = (_Float16)v;
        reinterpret_cast<uint16_t *>(n.wmc)[q] = *reinterpret_cast<const uint16_t *>(&hv);
    }
}

__device__ inline int cnn_nbr(int s, int k, int L);

// nbr[site][16]: neighbours 0, 2, 4, 6, 8 of the 3 x 3 window, three pads, neighbours 1, 3, 5, 7, four pads (the
// last neighbour again), as site numbers
__global__ void cnn_build_nbr_kernel(uint16_t *nbr, int L)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= L * L * 16) return;
    const int s = q >> 4, j = q & 7, odd = (q >> 3) & 1;
    nbr[q] = (uint16_t)cnn_nbr(s, min(2 * j + odd, 8), L);
}

nqs_status cnn_build_copy(nqs_model *m, int dtype, hipStream_t stream)
{
    const nqs_model_desc &d = m->desc;
    if (dtype == NQS_FP8_E4M3) return set_error(NQS_EUNSUPPORTED, "FP8 copies of the convolutional network are not built");
    Copy &c = m->copies[dtype];
    CnnDev &n = c.cnn;
    n.L = d.lat_L;
    n.F = d.widths[0];
    n.R = d.n_layers;
    n.dtype = dtype;
    const int F = n.F;
    CnnSeg segs[8 * NQS_MAX_LAYERS + 8];
    int ns = 0;
    int64_t off = 0;
    auto seg = [&](int64_t len, int conv) {
        segs[ns++] = CnnSeg{off, len, conv, F};
        const int64_t at = off;
        off += len;
        return at;
    };
    n.w0 = seg(9 * (int64_t)F, 1);
    n.b0 = seg(F, 0);
    for (int r = 0; r < n.R; ++r) {
        n.g[r] = seg(F, 0);
        n.be[r] = seg(F, 0);
        n.w1[r] = seg(9 * (int64_t)F * F, F);
        n.b1[r] = seg(F, 0);
        n.w2[r] = seg(9 * (int64_t)F * F, F);
        n.b2[r] = seg(F, 0);
    }
    n.gf = seg(F, 0);
    n.bef = seg(F, 0);
    if (off != m->P) return set_error(NQS_EINVAL, "convolutional network parameter count mismatch");
    const size_t pbytes = (sizeof(float) * (size_t)m->P + 255) & ~(size_t)255;
    const int64_t nmc = 2 * (int64_t)n.R * 9 * F * F;
    const size_t mfbytes = (sizeof(float) * (size_t)nmc + 255) & ~(size_t)255;
    const size_t mcbytes = dtype == NQS_F32 ? 0 : (sizeof(uint16_t) * (size_t)nmc + 255) & ~(size_t)255;
    const size_t sbytes = (sizeof(segs) + 255) & ~(size_t)255;
    if (!c.block) NQS_HIP_TRY(hipMalloc(&c.block, pbytes + sbytes + mfbytes + mcbytes + 32 * (size_t)n.L * n.L));
    n.p = (float *)c.block;
    CnnSeg *dsegs = (CnnSeg *)((char *)c.block + pbytes);
    n.wmf = (float *)((char *)c.block + pbytes + sbytes);
    n.wmc = dtype == NQS_F32 ? (void *)n.wmf : (void *)((char *)c.block + pbytes + sbytes + mfbytes);
    n.nbr = (uint16_t *)((char *)c.block + pbytes + sbytes + mfbytes + mcbytes);
    NQS_HIP_TRY(hipMemcpyAsync(dsegs, segs, sizeof(CnnSeg) * ns, hipMemcpyHostToDevice, stream));
    hipLaunchKernelGGL(cnn_build_kernel, dim3((unsigned)((m->P + 255) / 256)), dim3(256), 0, stream, m->master, m->P,
                       dtype, dsegs, ns, n.p);
    NQS_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(cnn_build_nbr_kernel, dim3((unsigned)((16 * n.L * n.L + 255) / 256)), dim3(256), 0, stream, n.nbr,
                       n.L);
    NQS_HIP_TRY(hipGetLastError());
    if (nmc > 0) {
        hipLaunchKernelGGL(cnn_build_mc_kernel, dim3((unsigned)((nmc + 255) / 256)), dim3(256), 0, stream, n, nmc);
        NQS_HIP_TRY(hipGetLastError());
    }
    // the host array of segments must outlive the copy
    NQS_HIP_TRY(hipStreamSynchronize(stream));
    c.valid = true;
    return NQS_OK;
}

// ---- the forward pass of one configuration by one workgroup ----

struct CnnLds {
    float *x;     // [S] spins
    float *h;     // [S][F] residual stream
    float *t;     // [S][F] phi(LN(h)), rounded
    float *u;     // [S][F] phi(conv1), rounded
    float *red;   // [kCnnThreads / 64]
};

__host__ __device__ inline size_t cnn_lds_bytes(int S, int F)
{
    return sizeof(float) * ((size_t)S + 3 * (size_t)S * F + kCnnThreads / 64);
}

__device__ inline CnnLds cnn_carve(float *sm, int S, int F)
{
    CnnLds l;
    l.x = sm;
    l.h = sm + S;
    l.t = l.h + (size_t)S * F;
    l.u = l.t + (size_t)S * F;
    l.red = l.u + (size_t)S * F;
    return l;
}

__device__ inline int cnn_nbr(int s, int k, int L)
{
    const int x = s / L, y = s - (s / L) * L;
    int xx = x + k / 3 - 1, yy = y + k % 3 - 1;
    xx += xx < 0 ? L : (xx >= L ? -L : 0);
    yy += yy < 0 ? L : (yy >= L ? -L : 0);
    return xx * L + yy;
}

__device__ inline float cnn_gelu(float x)
{
    const float c = 0.7978845608028654f;   // sqrt(2 / pi)
    return 0.5f * x * (1.0f + tanhf(c * fmaf(0.044715f * x * x, x, x)));
}

// FP32 -> format -> FP32, round to nearest even: BF16 by rounding the low 16
// bits of the encoding (same exponent range; NaN kept quiet), FP16 by the
// hardware conversion (round to nearest even, overflow to infinity).
__device__ inline float cnn_round(float v, int dtype)
{
    if (dtype == kBF16) {
        uint32_t u = __float_as_uint(v);
        if ((u & 0x7fffffffu) > 0x7f800000u) return __uint_as_float(u | 0x00400000u);
        u += 0x7fffu + ((u >> 16) & 1u);
        return __uint_as_float(u & 0xffff0000u);
    }
    if (dtype == kF16) return (float)(_Float16)v;
    return v;
}

// out[s][o] (+)= b[o] + sum_{k, c} W[c][k][o] in[nbr(s, k)][c]
__device__ inline float cnn_conv_at(const float *__restrict__ W, const float *__restrict__ b, const float *in, int s,
                                    int o, int L, int C, int F)
{
    float acc = b[o];
    for (int k = 0; k < 9; ++k) {
        const float *src = in + (size_t)cnn_nbr(s, k, L) * C;
        const float *w = W + (size_t)k * F + o;
        for (int c = 0; c < C; ++c) acc = fmaf(w[(size_t)c * 9 * F], src[c], acc);
    }
    return acc;
}

// log psi of the configuration in l.x (all threads return it); ends with a barrier
__device__ float cnn_forward(const CnnDev &net, const CnnLds &l)
{
    const int L = net.L, S = L * L, F = net.F, tid = threadIdx.x;
    const float *P = net.p;
    for (int idx = tid; idx < S * F; idx += kCnnThreads) {
        const int s = idx / F, o = idx - (idx / F) * F;
        l.h[idx] = cnn_conv_at(P + net.w0, P + net.b0, l.x, s, o, L, 1, F);
    }
    __syncthreads();
    for (int r = 0; r < net.R; ++r) {
        const float *g = P + net.g[r], *be = P + net.be[r];
        for (int s = tid; s < S; s += kCnnThreads) {
            const float *hs = l.h + (size_t)s * F;
            float mu = 0.0f;
            for (int c = 0; c < F; ++c) mu += hs[c];
            mu /= (float)F;
            float var = 0.0f;
            for (int c = 0; c < F; ++c) var = fmaf(hs[c] - mu, hs[c] - mu, var);
            const float rs = 1.0f / sqrtf(var / (float)F + kLnEps);
            for (int c = 0; c < F; ++c)
                l.t[(size_t)s * F + c] = cnn_round(cnn_gelu(fmaf((hs[c] - mu) * rs, g[c], be[c])), net.dtype);
        }
        __syncthreads();
        for (int idx = tid; idx < S * F; idx += kCnnThreads) {
            const int s = idx / F, o = idx - (idx / F) * F;
            l.u[idx] = cnn_round(cnn_gelu(cnn_conv_at(P + net.w1[r], P + net.b1[r], l.t, s, o, L, F, F)), net.dtype);
        }
        __syncthreads();
        for (int idx = tid; idx < S * F; idx += kCnnThreads) {
            const int s = idx / F, o = idx - (idx / F) * F;
            l.h[idx] += cnn_conv_at(P + net.w2[r], P + net.b2[r], l.u, s, o, L, F, F);
        }
        __syncthreads();
    }
    const float *g = P + net.gf, *be = P + net.bef;
    float part = 0.0f;
    for (int s = tid; s < S; s += kCnnThreads) {
        const float *hs = l.h + (size_t)s * F;
        float mu = 0.0f;
        for (int c = 0; c < F; ++c) mu += hs[c];
        mu /= (float)F;
        float var = 0.0f;
        for (int c = 0; c < F; ++c) var = fmaf(hs[c] - mu, hs[c] - mu, var);
        const float rs = 1.0f / sqrtf(var / (float)F + kLnEps);
        for (int c = 0; c < F; ++c) part += fmaf((hs[c] - mu) * rs, g[c], be[c]);
    }
    part = group_sum<64>(part);
    if ((tid & 63) == 0) l.red[tid >> 6] = part;
    __syncthreads();
    float f = 0.0f;
    for (int w = 0; w < kCnnThreads / 64; ++w) f += l.red[w];
    __syncthreads();
    return f;
}

// ---- log psi of given configurations ----

__global__ void __launch_bounds__(kCnnThreads) cnn_logpsi_kernel(CnnDev net, const int8_t *__restrict__ samples,
                                                                 int64_t n, float *__restrict__ logpsi)
{
    extern __shared__ float sm[];
    const int S = net.L * net.L;
    const CnnLds l = cnn_carve(sm, S, net.F);
    for (int64_t k = blockIdx.x; k < n; k += gridDim.x) {
        for (int i = threadIdx.x; i < S; i += kCnnThreads) l.x[i] = (float)samples[k * S + i];
        __syncthreads();
        const float f = cnn_forward(net, l);
        if (threadIdx.x == 0) logpsi[k] = f;
    }
}

// ---- Metropolis-Hastings, single flips, one chain per workgroup ----

struct CnnSampleArgs {
    CnnDev net;
    int8_t *chain_state;
    int8_t *samples;
    float *logpsi;
    unsigned long long *n_acc;
    int64_t n_chains;
    int n_sweeps, n_burnin, sweep_size;
    uint64_t seed, step_offset;
    uint32_t inst, chain_id_offset;
    int n_traced;
    int32_t *tr_site;
    uint32_t *tr_ubits;
    float *tr_delta;
    uint8_t *tr_acc;
};

__global__ void __launch_bounds__(kCnnThreads) cnn_sample_kernel(CnnSampleArgs A)
{
    extern __shared__ float sm[];
    __shared__ int s_site;
    __shared__ int s_accept;
    const int S = A.net.L * A.net.L, tid = threadIdx.x;
    const CnnLds l = cnn_carve(sm, S, A.net.F);
    const uint32_t key0 = (uint32_t)A.seed, key1 = (uint32_t)(A.seed >> 32);
    const int64_t total = (int64_t)(A.n_burnin + A.n_sweeps) * A.sweep_size;
    for (int64_t c = blockIdx.x; c < A.n_chains; c += gridDim.x) {
        const uint32_t gid = A.chain_id_offset + (uint32_t)c;
        for (int i = tid; i < S; i += kCnnThreads) l.x[i] = (float)A.chain_state[c * S + i];
        __syncthreads();
        float f = cnn_forward(A.net, l);
        unsigned long long acc = 0;
        for (int64_t k = 0; k < total; ++k) {
            const uint64_t step = A.step_offset + (uint64_t)k;
            uint32_t ub = 0;
            if (tid == 0) {
                const Block4 rb = philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), gid, A.inst << 8, key0, key1);
                s_site = index_from_word(rb.r0, S);
                ub = rb.r2 >> 8;
                l.x[s_site] = -l.x[s_site];
            }
            __syncthreads();
            const float fn = cnn_forward(A.net, l);
            if (tid == 0) {
                const float d = 2.0f * (fn - f);
                const float l2u = __builtin_amdgcn_logf((float)ub * 5.9604644775390625e-8f);   // log2 u
                const bool accept = l2u < d * 1.4426950408889634f;                            // NaN rejects
                s_accept = accept ? 1 : 0;
                if (!accept) l.x[s_site] = -l.x[s_site];
                if (c < A.n_traced) {
                    const size_t idx = (size_t)c * (size_t)total + (size_t)k;
                    A.tr_site[idx] = s_site | (0xFFFF << 16);
                    A.tr_ubits[idx] = ub;
                    A.tr_delta[idx] = d;
                    A.tr_acc[idx] = accept ? 1 : 0;
                }
            }
            __syncthreads();
            if (s_accept) {
                f = fn;
                ++acc;
            }
            if ((k + 1) % A.sweep_size == 0) {
                const int64_t out = (k + 1) / A.sweep_size - 1 - A.n_burnin;
                if (out >= 0) {
                    if (A.samples)
                        for (int i = tid; i < S; i += kCnnThreads)
                            A.samples[((size_t)out * A.n_chains + c) * S + i] = l.x[i] > 0.0f ? 1 : -1;
                    if (A.logpsi && tid == 0) A.logpsi[(size_t)out * A.n_chains + c] = f;
                    __syncthreads();   // the next proposal modifies l.x
                }
            }
        }
        for (int i = tid; i < S; i += kCnnThreads) A.chain_state[c * S + i] = l.x[i] > 0.0f ? 1 : -1;
        if (A.n_acc && tid == 0) A.n_acc[c] = acc;
        __syncthreads();
    }
}

// ---- TFIM local energies on the network's lattice, one sample per workgroup ----

__global__ void __launch_bounds__(kCnnThreads) cnn_eloc_tfim_kernel(CnnDev net, const int8_t *__restrict__ samples,
                                                                    int64_t n, double J, double h,
                                                                    double *__restrict__ eloc)
{
    extern __shared__ float sm[];
    const int L = net.L, S = L * L, tid = threadIdx.x;
    const CnnLds l = cnn_carve(sm, S, net.F);
    for (int64_t k = blockIdx.x; k < n; k += gridDim.x) {
        for (int i = tid; i < S; i += kCnnThreads) l.x[i] = (float)samples[k * S + i];
        __syncthreads();
        const float f0 = cnn_forward(net, l);
        double off = 0.0;
        for (int i = 0; i < S; ++i) {
            if (tid == 0) l.x[i] = -l.x[i];
            __syncthreads();
            const float fi = cnn_forward(net, l);
            off += exp((double)(fi - f0));
            if (tid == 0) l.x[i] = -l.x[i];
            __syncthreads();
        }
        if (tid == 0) {
            double diag = 0.0;
            for (int s = 0; s < S; ++s) {
                const int x = s / L, y = s - (s / L) * L;
                const int right = ((x + 1) % L) * L + y, down = x * L + (y + 1) % L;
                diag += (double)(l.x[s] * l.x[right]) + (double)(l.x[s] * l.x[down]);
            }
            eloc[k] = fma(h, off, J * diag);
        }
        __syncthreads();
    }
}

// ---- batched forward pass: B configurations per workgroup, convolutions on the matrix cores ----
//
// The forward pass of the B configurations of a workgroup (proposals of B chains, or B configurations of the
// local energies) is one batch of B * S rows (row = configuration x site).  Each convolution is the transposed
// product D[out channel][row] = W[out][9 F] in^T[9 F][row] over 16 x 16 tiles, its im2col operand gathered from
// LDS: v_mfma_f32_16x16x32_bf16 / _f16 (32 of the 9 F products per step) for 16-bit activations,
// v_mfma_f32_16x16x4_f32 (4 channels of one offset) for FP32 ones, FP32 accumulation.  A lane then holds four
// consecutive channels of one row, so the residual stream, the GELU outputs and their stores move 16 (8) bytes
// at a time, and a wave keeps the weights of its 16 output channels in registers for all of its tiles.
//
// What bounds it: the vector instructions of GELU (tanhf: about 45 per value, 2 R per site and channel) and of
// the layer norms; the products are 5 % of the time.  Hence
//   - 512 threads and at most 80 KB of LDS per workgroup, so that a CU runs two workgroups (four waves per
//     SIMD) and one's barriers and LDS round trips are filled by the other (the form with 256 threads and 105 KB
//     left one wave per SIMD);
//   - a layer norm's statistics are formed by one thread per row with 16-byte reads, and the GELU values by all
//     threads, four channels each (one thread per row for both read LDS with a stride of F words, 32 lanes on
//     one bank, and left 28 % of the threads idle for a 10 x 10 lattice).
// 10 x 10 lattice, 16 filters, 4 blocks, one sweep of 4096 chains, BF16: 26.0 ms with 256 threads and one thread
// per row, 13.2 ms in this form with GELU by tanhf, 6.7 ms now (vector instructions issue in 77 % of the cycles).
// Local energies of 1000 samples of it, FP32: 61.9 ms with one configuration per workgroup and each convolution
// output a chain of FMAs on operands from LDS and L2, 4.9 ms now.
//
// BIAS_FIRST starts each sum at the bias (v_mfma_f32_16x16x4_f32 adds its products one after another, each with
// one rounding, so the sum is the one-configuration kernel's chain of fmaf bit for bit); otherwise the bias is
// added to the finished sum.

typedef __bf16 cnn_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 cnn_h16x8 __attribute__((ext_vector_type(8)));
typedef float cnn_f32x4 __attribute__((ext_vector_type(4)));

// uniform reads of the parameters go through the scalar cache
typedef const float __attribute__((address_space(4))) cnn_cfloat;
__device__ __forceinline__ const cnn_cfloat *cnn_uniform(const float *p)
{
    return (const cnn_cfloat *)(uintptr_t)p;
}

constexpr int kMcThreads = 512;
constexpr int kMcWaves = kMcThreads / 64;

template <int DT> struct CnnMcT { typedef uint16_t E; };   // activations in LDS: raw codes
template <> struct CnnMcT<kF32> { typedef float E; };      // FP32 (rounded to the copy's format by the caller's `rnd`)

// phi(v) rounded to the 16-bit format DT, as its code: exactly round(cnn_gelu(v)) (binary16: its last product rounded
// once), at a third of its instructions.
// phi(x) = x / (1 + e), e = exp(-2 sqrt(2 / pi) (x + 0.044715 x^3)), takes one exponential and one reciprocal.
// Its error and that of the tanhf form are both below d = 1 + e units in the last place of the result (the tanhf
// form loses digits where 1 + tanh cancels, as d grows), so the two round to the same code unless the result lies
// within 4 d units of a rounding boundary; those values (about 1 in 1000 for BF16, and FP16's subnormal results)
// are formed by tanhf again.  Compared over all 2^32 inputs: equal codes for a bound of 2 d and above.
template <int DT>
__device__ __forceinline__ uint16_t cnn_gelu_code(float x)
{
    const float e = __builtin_amdgcn_exp2f(x * fmaf(x * x, -0.10294324f, -2.3022082f));
    const float d = 1.0f + e;
    float r = x * __builtin_amdgcn_rcpf(d);
    constexpr int kDrop = DT == kBF16 ? 16 : 13;
    const int off = (int)(__float_as_uint(r) & ((1u << kDrop) - 1u)) - (1 << (kDrop - 1));
    bool sure = fabsf((float)off) > 4.0f * d;
    if constexpr (DT == kF16) sure = sure && fabsf(r) >= 6.2e-5f;
    if constexpr (DT == kBF16) {
        if (!sure) r = cnn_gelu(x);
        const __bf16 c = (__bf16)r;       // one hardware conversion, to nearest even, NaN kept quiet
        return __builtin_bit_cast(uint16_t, c);
    } else {
        uint32_t c = __builtin_bit_cast(uint16_t, (_Float16)r);
        if (!sure) {
            // the last product of cnn_gelu rounded once, to binary16 (what the compiler makes of the product and a
            // conversion where it sees both)
            const float h = 0.5f * x, t = 1.0f + tanhf(0.7978845608028654f * fmaf(0.044715f * x * x, x, x));
            asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(c) : "v"(h), "v"(t));
        }
        return (uint16_t)c;
    }
}

// phi(v) of four consecutive channels 4 q .. 4 q + 3 of a row of activations, stored in the order the products read:
// 16-bit rows in channel order, FP32 rows with channel c at (c % 4) F / 4 + c / 4 (a lane's operands, the
// channels lk, lk + 4, ..., are then consecutive words)
template <int DT, int F>
__device__ __forceinline__ void cnn_mc_gelu4(typename CnnMcT<DT>::E *row, int q, const float *v, int rnd)
{
    if constexpr (DT == kF32) {
#pragma unroll
        for (int r = 0; r < 4; ++r) row[r * (F / 4) + q] = cnn_round(cnn_gelu(v[r]), rnd);
    } else {
        ushort4 c;
        c.x = cnn_gelu_code<DT>(v[0]);
        c.y = cnn_gelu_code<DT>(v[1]);
        c.z = cnn_gelu_code<DT>(v[2]);
        c.w = cnn_gelu_code<DT>(v[3]);
        *reinterpret_cast<ushort4 *>(row + 4 * q) = c;
    }
}

// LDS of a batch: residual stream, the two activation buffers, the spins, and per-configuration words of the
// callers
template <int F> struct CnnMcLds {
    float *h;            // [rows][F]
    void *t, *u;         // [rows][F] activations; the head of a row of t also holds its layer-norm statistics
    int8_t *x;           // [rows] spins
    float *w;            // per-configuration words
};

__host__ __device__ inline size_t cnn_mc_lds_bytes(int B, int S, int F, int esz)
{
    const size_t rows = (size_t)B * S;
    return rows * (sizeof(float) * F + 2 * (size_t)esz * F) + ((rows + 15) & ~(size_t)15) + 16 * (size_t)B;
}

template <int DT, int F>
__device__ __forceinline__ CnnMcLds<F> cnn_mc_carve(unsigned char *sm, int rows)
{
    typedef typename CnnMcT<DT>::E E;
    CnnMcLds<F> l;
    l.h = reinterpret_cast<float *>(sm);
    E *t = reinterpret_cast<E *>(l.h + (size_t)rows * F);
    l.t = t;
    l.u = t + (size_t)rows * F;
    l.x = reinterpret_cast<int8_t *>(t + 2 * (size_t)rows * F);
    l.w = reinterpret_cast<float *>(l.x + ((rows + 15) & ~15));
    return l;
}

// one convolution of the batch: u = phi(conv(in)) in the activation format, or h += conv(in).  s0: the site of
// this lane's row in its wave's first tile.  The gather's row numbers come from the copy's neighbour table (a few
// KB in the vector L1), read one tile ahead: forming them from (x, y) took a third of the vector instructions.
template <int DT, int F, bool RESID, bool BIAS_FIRST>
__device__ __forceinline__ void cnn_mc_conv(const typename CnnMcT<DT>::E *in, const void *wmc, const float *bias,
                                            int rows, int S, const uint16_t *nbr, int s0,
                                            typename CnnMcT<DT>::E *out, float *h, int rnd)
{
    typedef typename CnnMcT<DT>::E E;
    static_assert(F == 16 || F == 32, "16 or 32 channels");
    constexpr int NT = F / 16;                            // tiles of 16 output channels; a wave keeps one
    constexpr int kSteps = (9 * F + 31) / 32;             // 32-deep steps of the 16-bit forms
    constexpr bool kHalf = DT != kF32 && F == 16;         // a lane reads every other neighbour
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, la = lane & 15, lk = lane >> 4;
    const int nt = wave % NT, q = 4 * nt + lk;            // this lane's output channels: 4 q .. 4 q + 3
    const E *W = reinterpret_cast<const E *>(wmc);
    const float4 bq = *reinterpret_cast<const float4 *>(bias + 4 * q);
    const float b4[4] = {bq.x, bq.y, bq.z, bq.w};
    // step st of the 16-bit forms: F = 32, offset st, channels 8 lk .. 8 lk + 7; F = 16, offset 2 st + lk / 2,
    // channels 8 (lk % 2) .. + 7 (offset 9 of the last step has zero weights)
    const int c = DT == kF32 ? lk * (F / 4) : F == 32 ? 8 * lk : 8 * (lk & 1), hi = kHalf ? lk >> 1 : 0;
    constexpr int NW = DT == kF32 ? 9 * (F / 16) : kSteps;
    uint4 w[NW];
    if constexpr (DT == kF32) {
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int p = 0; p < F / 16; ++p)
                w[k * (F / 16) + p] =
                    *reinterpret_cast<const uint4 *>(W + ((size_t)k * F + nt * 16 + la) * F + c + 4 * p);
    } else {
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            const int k = F == 32 ? st : min(2 * st + hi, 8);
            w[st] = *reinterpret_cast<const uint4 *>(W + ((size_t)k * F + nt * 16 + la) * F + c);
            if (kHalf && 2 * st + hi > 8) w[st] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    constexpr int kStride = 16 * (kMcWaves / NT);         // rows from one of the wave's tiles to the next
    const int inc = kStride % S;
    int s = s0, row = wave / NT * 16 + la;
    // neighbours of this tile and the next
    auto load = [&](int site, uint4 &lo, uint4 &up) {
        const uint4 *tp = reinterpret_cast<const uint4 *>(nbr) + 2 * site;
        lo = tp[hi];
        if constexpr (!kHalf) up = tp[1];
    };
    uint4 lo, up = make_uint4(0u, 0u, 0u, 0u);
    load(s, lo, up);
    for (int r0 = wave / NT * 16; r0 < rows; r0 += kStride, row += kStride) {
        const bool live = row < rows;
        // rows past the last repeat the last configuration's sites
        const E *base = in + (size_t)(live ? row - s : rows - S) * F + c;
        const uint32_t pe[4] = {lo.x, lo.y, lo.z, lo.w}, po[4] = {up.x, up.y, up.z, up.w};
        int n[9];
#pragma unroll
        for (int k = 0; k < (kHalf ? kSteps : 9); ++k) {
            const int j = kHalf ? k : k >> 1;
            const uint32_t v = !kHalf && (k & 1) ? po[j >> 1] : pe[j >> 1];
            n[k] = (int)(j & 1 ? v >> 16 : v & 0xffffu);
        }
        s += inc;
        s = s >= S ? s - S : s;
        load(s, lo, up);
        cnn_f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (BIAS_FIRST) acc = cnn_f32x4{b4[0], b4[1], b4[2], b4[3]};
        if constexpr (DT == kF32) {
#pragma unroll
            for (int k = 0; k < 9; ++k) {
#pragma unroll
                for (int p = 0; p < F / 16; ++p) {
                    const float4 av = *reinterpret_cast<const float4 *>(base + n[k] * F + 4 * p);
                    const uint4 wv = w[k * (F / 16) + p];
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wv.x), av.x, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wv.y), av.y, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wv.z), av.z, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wv.w), av.w, acc, 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int st = 0; st < kSteps; ++st) {
                const uint4 av = *reinterpret_cast<const uint4 *>(base + n[st] * F);
                if constexpr (DT == kBF16) {
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(cnn_bf16x8, w[st]),
                                                                  __builtin_bit_cast(cnn_bf16x8, av), acc, 0, 0, 0);
                } else {
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(cnn_h16x8, w[st]),
                                                                 __builtin_bit_cast(cnn_h16x8, av), acc, 0, 0, 0);
                }
            }
        }
        // D[i][j] of a 16 x 16 block: j = lane % 16 (row), i = 4 (lane / 16) + register (output channel)
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = BIAS_FIRST ? acc[r] : acc[r] + b4[r];
        if (live) {
            if constexpr (RESID) {
                float4 *hp = reinterpret_cast<float4 *>(h + (size_t)row * F + 4 * q);
                float4 hv = *hp;
                hv.x += v[0];
                hv.y += v[1];
                hv.z += v[2];
                hv.w += v[3];
                *hp = hv;
            } else {
                cnn_mc_gelu4<DT, F>(out + (size_t)row * F, q, v, rnd);
            }
        }
    }
}

// mean and 1 / sqrt(var + eps) of a row's channels, summed in channel order
template <int F>
__device__ __forceinline__ void cnn_mc_stats(const float *hs, float &mu, float &rs)
{
    mu = 0.0f;
#pragma unroll
    for (int c = 0; c < F; ++c) mu += hs[c];
    mu /= (float)F;
    float var = 0.0f;
#pragma unroll
    for (int c = 0; c < F; ++c) var = fmaf(hs[c] - mu, hs[c] - mu, var);
    rs = 1.0f / sqrtf(var / (float)F + kLnEps);
}

// Forward pass of the configurations in l.x.  Leaves each row's sum over channels of the final layer norm in the
// first word of its row of t, and ends with a barrier.  `wmc`: the convolutions' operands for DT, 2 R blocks of
// 9 F^2; `rnd`: the format that activations are rounded to.
template <int DT, int F, bool BIAS_FIRST>
__device__ __forceinline__ void cnn_mc_forward(const CnnDev &net, const void *wmc, const CnnMcLds<F> &l, int rows,
                                               int rnd)
{
    typedef typename CnnMcT<DT>::E E;
    const int L = net.L, S = L * L, tid = threadIdx.x;
    const float *P = net.p;
    E *t = reinterpret_cast<E *>(l.t), *u = reinterpret_cast<E *>(l.u);
    const E *W = reinterpret_cast<const E *>(wmc);
    constexpr int64_t per = 9 * (int64_t)F * F;
    // embedding, one row per thread (the weights are uniform), and the first block's statistics
    const cnn_cfloat *w0 = cnn_uniform(P + net.w0), *b0 = cnn_uniform(P + net.b0);
    for (int row = tid; row < rows; row += kMcThreads) {
        const int s = row % S;
        const uint4 *np = reinterpret_cast<const uint4 *>(net.nbr) + 2 * s;
        const uint4 e = np[0], o = np[1];
        const int8_t *xb = l.x + (row - s);
        const float xv[9] = {(float)xb[e.x & 0xffffu], (float)xb[o.x & 0xffffu], (float)xb[e.x >> 16],
                             (float)xb[o.x >> 16],     (float)xb[e.y & 0xffffu], (float)xb[o.y & 0xffffu],
                             (float)xb[e.y >> 16],     (float)xb[o.y >> 16],     (float)xb[e.z & 0xffffu]};
        float hs[F];
#pragma unroll
        for (int o = 0; o < F; ++o) hs[o] = b0[o];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
#pragma unroll
            for (int o = 0; o < F; ++o) hs[o] = fmaf(w0[k * F + o], xv[k], hs[o]);
        }
#pragma unroll
        for (int o = 0; o < F; o += 4)
            *reinterpret_cast<float4 *>(l.h + (size_t)row * F + o) = make_float4(hs[o], hs[o + 1], hs[o + 2], hs[o + 3]);
        float2 st;
        cnn_mc_stats<F>(hs, st.x, st.y);
        *reinterpret_cast<float2 *>(t + (size_t)row * F) = st;
    }
    __syncthreads();
    constexpr int Q = F / 4;
    const int q = tid % Q, s0 = ((tid >> 6) / (F / 16) * 16 + (tid & 15)) % S;
    for (int r = 0; r < net.R; ++r) {
        if (r > 0) {
            for (int row = tid; row < rows; row += kMcThreads) {
                float hs[F];
#pragma unroll
                for (int o = 0; o < F; o += 4)
                    *reinterpret_cast<float4 *>(hs + o) = *reinterpret_cast<const float4 *>(l.h + (size_t)row * F + o);
                float2 st;
                cnn_mc_stats<F>(hs, st.x, st.y);
                *reinterpret_cast<float2 *>(t + (size_t)row * F) = st;
            }
            __syncthreads();
        }
        // phi(LN h): four channels of a row per thread.  The Q threads of a row are lanes of one wave, which
        // reads the row's statistics before it writes the row.
        const float4 gv = *reinterpret_cast<const float4 *>(P + net.g[r] + 4 * q);
        const float4 ev = *reinterpret_cast<const float4 *>(P + net.be[r] + 4 * q);
        for (int row = tid / Q; row < rows; row += kMcThreads / Q) {
            const float2 st = *reinterpret_cast<const float2 *>(t + (size_t)row * F);
            const float4 hv = *reinterpret_cast<const float4 *>(l.h + (size_t)row * F + 4 * q);
            const float v[4] = {fmaf((hv.x - st.x) * st.y, gv.x, ev.x), fmaf((hv.y - st.x) * st.y, gv.y, ev.y),
                                fmaf((hv.z - st.x) * st.y, gv.z, ev.z), fmaf((hv.w - st.x) * st.y, gv.w, ev.w)};
            cnn_mc_gelu4<DT, F>(t + (size_t)row * F, q, v, rnd);
        }
        __syncthreads();
        cnn_mc_conv<DT, F, false, BIAS_FIRST>(t, W + (2 * r) * per, P + net.b1[r], rows, S, net.nbr, s0, u, l.h,
                                              rnd);
        __syncthreads();
        cnn_mc_conv<DT, F, true, BIAS_FIRST>(u, W + (2 * r + 1) * per, P + net.b2[r], rows, S, net.nbr, s0, u, l.h,
                                             rnd);
        __syncthreads();
    }
    const cnn_cfloat *gf = cnn_uniform(P + net.gf), *bef = cnn_uniform(P + net.bef);
    for (int row = tid; row < rows; row += kMcThreads) {
        float hs[F];
#pragma unroll
        for (int o = 0; o < F; o += 4)
            *reinterpret_cast<float4 *>(hs + o) = *reinterpret_cast<const float4 *>(l.h + (size_t)row * F + o);
        float mu, rs;
        cnn_mc_stats<F>(hs, mu, rs);
        float a = 0.0f;
#pragma unroll
        for (int c = 0; c < F; ++c) a += fmaf((hs[c] - mu) * rs, gf[c], bef[c]);
        *reinterpret_cast<float *>(t + (size_t)row * F) = a;
    }
    __syncthreads();
}

// ---- sampler on the batched forward pass: the B chains of a workgroup propose in lockstep ----

template <int DT, int F>
__global__ void __launch_bounds__(kMcThreads, 4) cnn_sample_mc_kernel(CnnSampleArgs A, int B)
{
    typedef typename CnnMcT<DT>::E E;
    extern __shared__ __align__(16) unsigned char smc[];
    const int L = A.net.L, S = L * L, rows = B * S, tid = threadIdx.x;
    const CnnMcLds<F> l = cnn_mc_carve<DT, F>(smc, rows);
    int8_t *x = l.x;
    const E *rsum = reinterpret_cast<const E *>(l.t);
    float *fcur = l.w;
    int *site = reinterpret_cast<int *>(fcur + B), *accn = site + B;
    uint32_t *ubs = reinterpret_cast<uint32_t *>(accn + B);
    const uint32_t key0 = (uint32_t)A.seed, key1 = (uint32_t)(A.seed >> 32);
    const int64_t total = (int64_t)(A.n_burnin + A.n_sweeps) * A.sweep_size;
    // log psi of configuration b from its rows' sums, in site order
    auto logpsi_of = [&](int b) {
        float a = 0.0f;
#pragma unroll 4
        for (int s = 0; s < S; ++s) a += *reinterpret_cast<const float *>(rsum + (size_t)(b * S + s) * F);
        return a;
    };
    for (int64_t c0 = (int64_t)blockIdx.x * B; c0 < A.n_chains; c0 += (int64_t)gridDim.x * B) {
        for (int i = tid; i < rows; i += kMcThreads) {
            const int64_t c = c0 + i / S;
            x[i] = c < A.n_chains ? A.chain_state[c * S + i % S] : (int8_t)1;
        }
        __syncthreads();
        cnn_mc_forward<DT, F, false>(A.net, A.net.wmc, l, rows, DT);
        // the thread of chain `tid` flips the site of proposal k
        auto propose = [&](int64_t k) {
            const uint64_t step = A.step_offset + (uint64_t)k;
            const uint32_t gid = A.chain_id_offset + (uint32_t)(c0 + tid);
            const Block4 rb = philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), gid, A.inst << 8, key0, key1);
            const int i = index_from_word(rb.r0, S);
            site[tid] = i;
            ubs[tid] = rb.r2 >> 8;
            x[tid * S + i] = (int8_t)-x[tid * S + i];
        };
        if (tid < B) {
            accn[tid] = 0;
            fcur[tid] = logpsi_of(tid);
            if (total > 0) propose(0);
        }
        __syncthreads();
        int64_t in_sweep = 0, out = -(int64_t)A.n_burnin;
        for (int64_t k = 0; k < total; ++k) {
            cnn_mc_forward<DT, F, false>(A.net, A.net.wmc, l, rows, DT);
            const bool sweep_end = ++in_sweep == A.sweep_size;
            if (tid < B) {
                const int64_t c = c0 + tid;
                const float fn = logpsi_of(tid);
                const float d = 2.0f * (fn - fcur[tid]);
                const float l2u = __builtin_amdgcn_logf((float)ubs[tid] * 5.9604644775390625e-8f);
                const bool accept = l2u < d * 1.4426950408889634f;
                if (accept) {
                    fcur[tid] = fn;
                    ++accn[tid];
                } else {
                    x[tid * S + site[tid]] = (int8_t)-x[tid * S + site[tid]];
                }
                if (c < A.n_traced) {
                    const size_t idx = (size_t)c * (size_t)total + (size_t)k;
                    A.tr_site[idx] = site[tid] | (0xFFFF << 16);
                    A.tr_ubits[idx] = ubs[tid];
                    A.tr_delta[idx] = d;
                    A.tr_acc[idx] = accept ? 1 : 0;
                }
                if (!sweep_end) propose(k + 1);
            }
            __syncthreads();
            if (sweep_end) {
                in_sweep = 0;
                if (out >= 0) {
                    for (int i = tid; i < rows; i += kMcThreads) {
                        const int64_t c = c0 + i / S;
                        if (c < A.n_chains && A.samples)
                            A.samples[((size_t)out * A.n_chains + c) * S + i % S] = x[i] > 0 ? 1 : -1;
                    }
                    if (A.logpsi && tid < B && c0 + tid < A.n_chains)
                        A.logpsi[(size_t)out * A.n_chains + c0 + tid] = fcur[tid];
                }
                ++out;
                if (k + 1 < total) {
                    __syncthreads();   // the next proposal modifies x
                    if (tid < B) propose(k + 1);
                    __syncthreads();
                }
            }
        }
        for (int i = tid; i < rows; i += kMcThreads) {
            const int64_t c = c0 + i / S;
            if (c < A.n_chains) A.chain_state[c * S + i % S] = x[i] > 0 ? 1 : -1;
        }
        if (A.n_acc && tid < B && c0 + tid < A.n_chains) A.n_acc[c0 + tid] = (unsigned long long)accn[tid];
        __syncthreads();
    }
}

// ---- TFIM local energies on the batched forward pass ----
//
// The n (S + 1) configurations (each sample, then its S flips) are numbered through and a workgroup takes B at a
// time, so that the grid is full whatever n is; their log psi go to f[n][S + 1] and one wave per sample sums the
// ratios.  FP32 products on the matrix cores for every format (activations rounded to it), each sum a chain of
// fmaf that starts at the bias, so the log psi are the one-configuration kernel's bit for bit.
template <int F>
__global__ void __launch_bounds__(kMcThreads, 4) cnn_eloc_logpsi_kernel(CnnDev net, const int8_t *__restrict__ samples,
                                                                        int64_t n, int B, float *__restrict__ f)
{
    extern __shared__ __align__(16) unsigned char smc[];
    const int L = net.L, S = L * L, rows = B * S, tid = threadIdx.x;
    const CnnMcLds<F> l = cnn_mc_carve<kF32, F>(smc, rows);
    const float *rsum = reinterpret_cast<const float *>(l.t);
    const int64_t total = n * (S + 1);
    for (int64_t q0 = (int64_t)blockIdx.x * B; q0 < total; q0 += (int64_t)gridDim.x * B) {
        for (int i = tid; i < rows; i += kMcThreads) {
            const int b = i / S, s = i - b * S;
            const int64_t q = q0 + b < total ? q0 + b : total - 1, k = q / (S + 1);
            const int flip = (int)(q - k * (S + 1)) - 1;
            const int8_t v = samples[k * S + s];
            l.x[i] = s == flip ? (int8_t)-v : v;
        }
        __syncthreads();
        cnn_mc_forward<kF32, F, true>(net, net.wmf, l, rows, net.dtype);
        // log psi in the one-configuration kernel's order: a site per thread, a wave's threads by a butterfly,
        // then the four waves
        const int lane = tid & 63;
        for (int b = tid >> 6; b < B; b += kMcWaves) {
            float a = 0.0f;
            for (int w = 0; w < kCnnThreads / 64; ++w) {
                const int s = w * 64 + lane;
                a += group_sum<64>(s < S ? rsum[(size_t)(b * S + s) * F] : 0.0f);
            }
            if (lane == 0 && q0 + b < total) f[q0 + b] = a;
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) cnn_eloc_reduce_kernel(const int8_t *__restrict__ samples,
                                                              const float *__restrict__ f, int64_t n, int L, double J,
                                                              double h, double *__restrict__ eloc)
{
    const int S = L * L, lane = threadIdx.x & 63;
    const int64_t k = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6);
    if (k >= n) return;
    const float *fk = f + k * (S + 1);
    const float f0 = fk[0];
    const int8_t *x = samples + k * S;
    double off = 0.0, diag = 0.0;
    for (int s0 = 0; s0 < S; s0 += 64) {
        const int s = s0 + lane;
        const double e = s < S ? exp((double)(fk[1 + s] - f0)) : 0.0;
        double d = 0.0;
        if (s < S) {
            const int sx = s / L, sy = s - sx * L;
            const int right = ((sx + 1) % L) * L + sy, down = sx * L + (sy + 1) % L;
            d = (double)(x[s] * x[right]) + (double)(x[s] * x[down]);
        }
        diag += group_sum<64>(d);            // whole numbers: exact in any order
        for (int i = 0; i < 64; ++i) off += __shfl(e, i, 64);   // site order (zeros past the last site)
    }
    if (lane == 0) eloc[k] = fma(h, off, J * diag);   // as the one-configuration kernel, to the last bit
}

// Whether the batched sampler serves this network (its log psi differs from the one-chain kernel's in the order
// of the sums, so the choice depends on the network alone).
static bool cnn_mc_applies(const CnnDev &net)
{
    if (net.F != 16 && net.F != 32) return false;
    const size_t S = (size_t)net.L * net.L, esz = net.dtype == NQS_F32 ? 4 : 2;
    for (size_t B : {16, 8, 4, 2, 1}) {
        const size_t rows = B * S;
        size_t b = (sizeof(float) * (rows + rows * net.F) + 15) & ~(size_t)15;
        b = (b + 2 * esz * rows * net.F + 15) & ~(size_t)15;
        if (rows % 16 == 0 && b + sizeof(float) * rows + 20 * B <= 160 * 1024) return true;
    }
    return false;
}

// Configurations per workgroup, at most 512 rows (four tiles of 16 for each of eight waves) within 80 KB of LDS
// (two workgroups per CU), or one configuration whatever it takes: the number that needs the fewest rounds x rows
// (+ 64 rows' worth of barriers and latency a pass) for `count` configurations.  10 x 10 lattice, 4096 chains: 4
// configurations fill two rounds; 5 need as many, with a quarter more rows each (10.4 ms at 5 and with the
// neighbours formed from (x, y), 6.7 ms at 4 and with their table).
static int cnn_mc_batch(int S, int F, int esz, int64_t count)
{
    int best = 1;
    double cost = 0.0;
    for (int B = 1; B == 1 || (B * S <= 512 && cnn_mc_lds_bytes(B, S, F, esz) <= 80 * 1024); ++B) {
        const int64_t slots = (cnn_mc_lds_bytes(B, S, F, esz) <= 80 * 1024 ? 2 : 1) * (int64_t)device_cus();
        const int64_t groups = (count + B - 1) / B, rounds = (groups + slots - 1) / slots;
        const double c = (double)rounds * (B * S + 64);
        if (B == 1 || c < cost) {
            best = B;
            cost = c;
        }
    }
    return best;
}

template <int DT>
static void launch_cnn_mc(const CnnSampleArgs &A, int B, int64_t blocks, size_t lds, hipStream_t stream)
{
    if (A.net.F == 16) {
        allow_lds(cnn_sample_mc_kernel<DT, 16>, lds);
        hipLaunchKernelGGL((cnn_sample_mc_kernel<DT, 16>), dim3((unsigned)blocks), dim3(kMcThreads), lds, stream, A, B);
    } else {
        allow_lds(cnn_sample_mc_kernel<DT, 32>, lds);
        hipLaunchKernelGGL((cnn_sample_mc_kernel<DT, 32>), dim3((unsigned)blocks), dim3(kMcThreads), lds, stream, A, B);
    }
}

// ---- host ----

static nqs_status cnn_check(const CnnDev &net)
{
    if (cnn_lds_bytes(net.L * net.L, net.F) > 160 * 1024)
        return set_error(NQS_EUNSUPPORTED, "convolutional network activations exceed 160 KB of LDS (L^2 x F too large)");
    return NQS_OK;
}

nqs_status cnn_logpsi(nqs_model *m, const int8_t *samples, int64_t n, float *logpsi, hipStream_t stream)
{
    nqs_status st = ensure_copy(m, NQS_F32, stream);
    if (st != NQS_OK) return st;
    const CnnDev &net = m->copies[NQS_F32].cnn;
    if ((st = cnn_check(net)) != NQS_OK) return st;
    const size_t lds = cnn_lds_bytes(net.L * net.L, net.F);
    allow_lds(cnn_logpsi_kernel, lds);
    const int64_t blocks = std::min<int64_t>(n, (int64_t)device_cus() * 16);
    hipLaunchKernelGGL(cnn_logpsi_kernel, dim3((unsigned)blocks), dim3(kCnnThreads), lds, stream, net, samples, n, logpsi);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

nqs_status cnn_sample(nqs_model *m, const nqs_sample_cfg &cfg, int8_t *chain_state, int8_t *samples, float *logpsi,
                      uint64_t *n_accepted, const nqs_trace *trace, hipStream_t stream)
{
    nqs_status st = ensure_copy(m, cfg.dtype, stream);
    if (st != NQS_OK) return st;
    const CnnDev &net = m->copies[cfg.dtype].cnn;
    if ((st = cnn_check(net)) != NQS_OK) return st;
    const int S = net.L * net.L;
    if (cfg.init_chains) {
        st = launch_init_chains(chain_state, cfg.n_chains, S, NQS_MOVE_FLIP, cfg.seed, cfg.instance_id,
                                cfg.chain_id_offset, stream);
        if (st != NQS_OK) return st;
    }
    CnnSampleArgs A;
    A.net = net;
    A.chain_state = chain_state;
    A.samples = samples;
    A.logpsi = logpsi;
    A.n_acc = (unsigned long long *)n_accepted;
    A.n_chains = cfg.n_chains;
    A.n_sweeps = cfg.n_sweeps;
    A.n_burnin = cfg.n_burnin;
    A.sweep_size = cfg.sweep_size > 0 ? cfg.sweep_size : S;
    A.seed = cfg.seed;
    A.step_offset = cfg.step_offset;
    A.inst = cfg.instance_id;
    A.chain_id_offset = (uint32_t)cfg.chain_id_offset;
    const bool tr = trace && trace->n_chains_traced > 0;
    A.n_traced = tr ? trace->n_chains_traced : 0;
    A.tr_site = tr ? trace->site : nullptr;
    A.tr_ubits = tr ? trace->ubits : nullptr;
    A.tr_delta = tr ? trace->delta : nullptr;
    A.tr_acc = tr ? trace->accepted : nullptr;
    if (cfg.lanes_per_chain != -1 && cnn_mc_applies(net)) {
        const int esz = net.dtype == NQS_F32 ? 4 : 2, B = cnn_mc_batch(S, net.F, esz, cfg.n_chains);
        const size_t lds = cnn_mc_lds_bytes(B, S, net.F, esz);
        const int64_t groups = (cfg.n_chains + B - 1) / B;
        const int64_t blocks = std::min<int64_t>(groups, (int64_t)device_cus() * 16);
        if (net.dtype == NQS_BF16) launch_cnn_mc<kBF16>(A, B, blocks, lds, stream);
        else if (net.dtype == NQS_F16) launch_cnn_mc<kF16>(A, B, blocks, lds, stream);
        else launch_cnn_mc<kF32>(A, B, blocks, lds, stream);
        NQS_HIP_TRY(hipGetLastError());
        return NQS_OK;
    }
    const size_t lds = cnn_lds_bytes(S, net.F);
    allow_lds(cnn_sample_kernel, lds);
    const int64_t blocks = std::min<int64_t>(cfg.n_chains, (int64_t)device_cus() * 16);
    hipLaunchKernelGGL(cnn_sample_kernel, dim3((unsigned)blocks), dim3(kCnnThreads), lds, stream, A);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

nqs_status cnn_local_energy(nqs_model *m, const nqs_ham_desc &ham, const int8_t *samples, int64_t n, int dtype,
                            double *eloc, hipStream_t stream)
{
    if (ham.kind != NQS_TFIM || ham.dim != 2 || ham.L != m->desc.lat_L || !ham.pbc)
        return set_error(NQS_EUNSUPPORTED,
                         "convolutional-network local energies: TFIM on the network's periodic L x L lattice");
    nqs_status st = ensure_copy(m, dtype, stream);
    if (st != NQS_OK) return st;
    const CnnDev &net = m->copies[dtype].cnn;
    if ((st = cnn_check(net)) != NQS_OK) return st;
    const int L = net.L, S = L * L, F = net.F;
    // 16 and 32 channels on up to 256 sites whose batch fits LDS: the batched forward pass, whose log psi are the
    // one-configuration kernel's bit for bit (beyond 256 sites a thread of that kernel sums two sites' channels as one
    // chain).  A captured call and one that gets no scratch take the one-configuration kernel, which needs none.
    if ((F == 16 || F == 32) && S <= kCnnThreads && cnn_mc_lds_bytes(1, S, F, 4) <= 160 * 1024 &&
        !stream_capturing(stream)) {
        const ScratchLease lease(stream);
        if (float *f = (float *)lease.ptr()) {
            // the samples whose log psi values the scratch holds
            const int64_t chunk = std::min<int64_t>(n, (int64_t)(kScratchBytes / sizeof(float)) / (S + 1));
            for (int64_t k0 = 0; k0 < n; k0 += chunk) {
                const int64_t kn = std::min(chunk, n - k0), count = kn * (S + 1);
                const int B = cnn_mc_batch(S, F, 4, count);
                const size_t lds = cnn_mc_lds_bytes(B, S, F, 4);
                const int64_t per_cu = lds <= 80 * 1024 ? 2 : 1;
                const int64_t blocks = std::min<int64_t>((count + B - 1) / B, per_cu * device_cus());
                auto launch = [&](auto kernel) {
                    allow_lds(kernel, lds);
                    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kMcThreads), lds, stream, net,
                                       samples + k0 * S, kn, B, f);
                };
                if (F == 16) launch(cnn_eloc_logpsi_kernel<16>);
                else launch(cnn_eloc_logpsi_kernel<32>);
                NQS_HIP_TRY(hipGetLastError());
                hipLaunchKernelGGL(cnn_eloc_reduce_kernel, dim3((unsigned)((kn + 3) / 4)), dim3(256), 0, stream,
                                   samples + k0 * S, f, kn, L, ham.J, ham.h, eloc + k0);
                NQS_HIP_TRY(hipGetLastError());
            }
            return NQS_OK;
        }
    }
    const size_t lds = cnn_lds_bytes(S, F);
    allow_lds(cnn_eloc_tfim_kernel, lds);
    const int64_t blocks = std::min<int64_t>(n, (int64_t)device_cus() * 16);
    hipLaunchKernelGGL(cnn_eloc_tfim_kernel, dim3((unsigned)blocks), dim3(kCnnThreads), lds, stream, net, samples, n,
                       ham.J, ham.h, eloc);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

// ---- log-derivatives O = d log psi / d theta (Eq. eq:forces), FP32 copy ----
//
// One sample per workgroup.  The forward pass keeps the residual stream before
// every block and after the last, each block's conv1 pre-activation and the
// layer-norm statistics in LDS; the backward pass recomputes phi(LN h) and
// phi(conv1) from them.  Every derivative is a fixed-order sum over sites.

__device__ inline float cnn_gelu_grad(float z)
{
    const float c = 0.7978845608028654f;
    const float a = c * fmaf(0.044715f * z * z, z, z);
    const float th = tanhf(a);
    return 0.5f * (1.0f + th) + 0.5f * z * (1.0f - th * th) * c * fmaf(3.0f * 0.044715f, z * z, 1.0f);
}

__host__ __device__ inline size_t cnn_grad_lds_bytes(int S, int F, int R)
{
    const size_t SF = (size_t)S * F;
    return sizeof(float) * ((size_t)S + (size_t)(2 * R + 1) * SF + 2 * (size_t)(R + 1) * S + 4 * SF +
                            kCnnThreads / 64);
}

// per-site layer-norm statistics of h into mu[s], rs[s]
__device__ inline void cnn_ln_stats(const float *h, int S, int F, float *mu, float *rs)
{
    for (int s = threadIdx.x; s < S; s += kCnnThreads) {
        const float *hs = h + (size_t)s * F;
        float m = 0.0f;
        for (int c = 0; c < F; ++c) m += hs[c];
        m /= (float)F;
        float v = 0.0f;
        for (int c = 0; c < F; ++c) v = fmaf(hs[c] - m, hs[c] - m, v);
        mu[s] = m;
        rs[s] = 1.0f / sqrtf(v / (float)F + kLnEps);
    }
}

// gh[s][:] += LN backward of gz (gradient at the layer-norm output) through scale g
__device__ inline void cnn_ln_back(const float *h, const float *mu, const float *rs, const float *gz, const float *g,
                                   int S, int F, float *gh)
{
    for (int s = threadIdx.x; s < S; s += kCnnThreads) {
        const float *hs = h + (size_t)s * F, *gs = gz + (size_t)s * F;
        float m1 = 0.0f, m2 = 0.0f;
        for (int c = 0; c < F; ++c) {
            const float gn = gs[c] * g[c];
            m1 += gn;
            m2 = fmaf(gn, (hs[c] - mu[s]) * rs[s], m2);
        }
        m1 /= (float)F;
        m2 /= (float)F;
        for (int c = 0; c < F; ++c) {
            const float gn = gs[c] * g[c], nh = (hs[c] - mu[s]) * rs[s];
            gh[(size_t)s * F + c] += rs[s] * (gn - m1 - nh * m2);
        }
    }
}

// O[off + (o*C + c)*9 + k] = sum_s g[s][o] in[nbr(s,k)][c];  O[boff + o] = sum_s g[s][o]
__device__ inline void cnn_wgrad(const float *g, const float *in, int S, int L, int C, int F, float *O, int64_t off,
                                 int64_t boff)
{
    const int n = 9 * C * F;
    for (int q = threadIdx.x; q < n + F; q += kCnnThreads) {
        if (q < n) {
            const int o = q / (9 * C), r = q - o * 9 * C, c = r / 9, k = r - c * 9;
            float a = 0.0f;
            for (int s = 0; s < S; ++s) a = fmaf(g[(size_t)s * F + o], in[(size_t)cnn_nbr(s, k, L) * C + c], a);
            O[off + q] = a;
        } else {
            const int o = q - n;
            float a = 0.0f;
            for (int s = 0; s < S; ++s) a += g[(size_t)s * F + o];
            O[boff + o] = a;
        }
    }
}

// gin[s'][c] = sum_{k,o} W[c][k][o] g[nbr(s', 8 - k)][o]   (the transposed convolution)
__device__ inline void cnn_inback(const float *__restrict__ W, const float *g, int S, int L, int F, float *gin)
{
    for (int idx = threadIdx.x; idx < S * F; idx += kCnnThreads) {
        const int s = idx / F, c = idx - (idx / F) * F;
        float a = 0.0f;
        for (int k = 0; k < 9; ++k) {
            const float *gs = g + (size_t)cnn_nbr(s, 8 - k, L) * F;
            const float *w = W + ((size_t)c * 9 + k) * F;
            for (int o = 0; o < F; ++o) a = fmaf(w[o], gs[o], a);
        }
        gin[idx] = a;
    }
}

__global__ void __launch_bounds__(kCnnThreads) cnn_grad_kernel(CnnDev net, const int8_t *__restrict__ samples,
                                                               int64_t n, int64_t P, float *__restrict__ logpsi,
                                                               float *__restrict__ O)
{
    extern __shared__ float sm[];
    const int L = net.L, S = L * L, F = net.F, R = net.R, tid = threadIdx.x;
    const size_t SF = (size_t)S * F;
    float *x = sm;
    float *H = x + S;                       // [R+1][S][F]
    float *A1 = H + (size_t)(R + 1) * SF;   // [R][S][F]
    float *MU = A1 + (size_t)R * SF;        // [R+1][S]
    float *RS = MU + (size_t)(R + 1) * S;   // [R+1][S]
    float *gh = RS + (size_t)(R + 1) * S;   // [S][F]
    float *gu = gh + SF;
    float *T1 = gu + SF;
    float *T2 = T1 + SF;
    float *red = T2 + SF;
    const float *Pp = net.p;
    for (int64_t row = blockIdx.x; row < n; row += gridDim.x) {
        float *Orow = O ? O + row * P : nullptr;
        for (int i = tid; i < S; i += kCnnThreads) x[i] = (float)samples[row * S + i];
        __syncthreads();
        // forward, keeping what the backward pass needs
        for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
            const int s = idx / F, o = idx - (idx / F) * F;
            H[idx] = cnn_conv_at(Pp + net.w0, Pp + net.b0, x, s, o, L, 1, F);
        }
        __syncthreads();
        for (int r = 0; r < R; ++r) {
            const float *h = H + (size_t)r * SF;
            cnn_ln_stats(h, S, F, MU + (size_t)r * S, RS + (size_t)r * S);
            __syncthreads();
            const float *g = Pp + net.g[r], *be = Pp + net.be[r];
            for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
                const int s = idx / F, c = idx - (idx / F) * F;
                T1[idx] = cnn_gelu(fmaf((h[idx] - MU[r * S + s]) * RS[r * S + s], g[c], be[c]));
            }
            __syncthreads();
            float *a1 = A1 + (size_t)r * SF;
            for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
                const int s = idx / F, o = idx - (idx / F) * F;
                const float a = cnn_conv_at(Pp + net.w1[r], Pp + net.b1[r], T1, s, o, L, F, F);
                a1[idx] = a;
                T2[idx] = cnn_gelu(a);
            }
            __syncthreads();
            float *hn = H + (size_t)(r + 1) * SF;
            for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
                const int s = idx / F, o = idx - (idx / F) * F;
                hn[idx] = h[idx] + cnn_conv_at(Pp + net.w2[r], Pp + net.b2[r], T2, s, o, L, F, F);
            }
            __syncthreads();
        }
        const float *hR = H + (size_t)R * SF;
        float *muR = MU + (size_t)R * S, *rsR = RS + (size_t)R * S;
        cnn_ln_stats(hR, S, F, muR, rsR);
        __syncthreads();
        const float *gf = Pp + net.gf, *bef = Pp + net.bef;
        float part = 0.0f;
        for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
            const int s = idx / F, c = idx - (idx / F) * F;
            part += fmaf((hR[idx] - muR[s]) * rsR[s], gf[c], bef[c]);
        }
        part = group_sum<64>(part);
        if ((tid & 63) == 0) red[tid >> 6] = part;
        __syncthreads();
        if (tid == 0 && logpsi) {
            float f = 0.0f;
            for (int w = 0; w < kCnnThreads / 64; ++w) f += red[w];
            logpsi[row] = f;
        }
        if (Orow) {
            // readout: d/d gamma_f, d/d beta_f; gradient at the final layer-norm output is 1
            for (int c = tid; c < F; c += kCnnThreads) {
                float a = 0.0f;
                for (int s = 0; s < S; ++s) a += (hR[(size_t)s * F + c] - muR[s]) * rsR[s];
                Orow[net.gf + c] = a;
                Orow[net.bef + c] = (float)S;
            }
            for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
                gu[idx] = 1.0f;
                gh[idx] = 0.0f;
            }
            __syncthreads();
            cnn_ln_back(hR, muR, rsR, gu, gf, S, F, gh);
            __syncthreads();
            for (int r = R - 1; r >= 0; --r) {
                const float *h = H + (size_t)r * SF, *a1 = A1 + (size_t)r * SF;
                const float *mu = MU + (size_t)r * S, *rs = RS + (size_t)r * S;
                const float *g = Pp + net.g[r], *be = Pp + net.be[r];
                for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
                    const int s = idx / F, c = idx - (idx / F) * F;
                    T1[idx] = cnn_gelu(fmaf((h[idx] - mu[s]) * rs[s], g[c], be[c]));   // t
                    T2[idx] = cnn_gelu(a1[idx]);                                        // u
                }
                __syncthreads();
                // conv2: weights from gh and u; gradient at u
                cnn_wgrad(gh, T2, S, L, F, F, Orow, net.w2[r], net.b2[r]);
                cnn_inback(Pp + net.w2[r], gh, S, L, F, gu);
                __syncthreads();
                for (int idx = tid; idx < (int)SF; idx += kCnnThreads) gu[idx] *= cnn_gelu_grad(a1[idx]);
                __syncthreads();
                // conv1: weights from the conv1 gradient and t; gradient at t (into T2)
                cnn_wgrad(gu, T1, S, L, F, F, Orow, net.w1[r], net.b1[r]);
                cnn_inback(Pp + net.w1[r], gu, S, L, F, T2);
                __syncthreads();
                // through phi and the block's layer norm (scale and shift), into gh
                for (int idx = tid; idx < (int)SF; idx += kCnnThreads) {
                    const int s = idx / F, c = idx - (idx / F) * F;
                    T2[idx] *= cnn_gelu_grad(fmaf((h[idx] - mu[s]) * rs[s], g[c], be[c]));
                }
                __syncthreads();
                for (int c = tid; c < F; c += kCnnThreads) {
                    float ag = 0.0f, ab = 0.0f;
                    for (int s = 0; s < S; ++s) {
                        const float gz = T2[(size_t)s * F + c];
                        ag = fmaf(gz, (h[(size_t)s * F + c] - mu[s]) * rs[s], ag);
                        ab += gz;
                    }
                    Orow[net.g[r] + c] = ag;
                    Orow[net.be[r] + c] = ab;
                }
                cnn_ln_back(h, mu, rs, T2, g, S, F, gh);
                __syncthreads();
            }
            cnn_wgrad(gh, x, S, L, 1, F, Orow, net.w0, net.b0);
        }
        __syncthreads();
    }
}

// vjp_out[p] += sum_k g[k] O[k][p] over a chunk of samples (FP64 accumulation per chunk)
__global__ void vjp_chunk_kernel(const float *__restrict__ O, const float *__restrict__ g, int64_t n, int64_t P,
                                 float *__restrict__ out, int first)
{
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    double acc = first ? 0.0 : (double)out[p];
    for (int64_t k = 0; k < n; ++k) acc += (double)g[k] * (double)O[k * P + p];
    out[p] = (float)acc;
}

static nqs_status launch_vjp_chunk(const float *O, const float *g, int64_t n, int64_t P, float *out, bool first,
                            hipStream_t stream)
{
    hipLaunchKernelGGL(vjp_chunk_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, stream, O, g, n, P, out,
                       first ? 1 : 0);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

nqs_status cnn_logpsi_grad(nqs_model *m, const int8_t *samples, int64_t n, float *logpsi, float *O,
                           const float *vjp_in, float *vjp_out, hipStream_t stream)
{
    nqs_status st = ensure_copy(m, NQS_F32, stream);
    if (st != NQS_OK) return st;
    const CnnDev &net = m->copies[NQS_F32].cnn;
    const int S = net.L * net.L;
    const size_t lds = cnn_grad_lds_bytes(S, net.F, net.R);
    if (lds > 160 * 1024)
        return set_error(NQS_EUNSUPPORTED, "convolutional-network gradient: activations exceed 160 KB of LDS");
    allow_lds(cnn_grad_kernel, lds);
    const int64_t P = m->P;
    if (logpsi || O) {
        const int64_t blocks = std::min<int64_t>(n, (int64_t)device_cus() * 16);
        hipLaunchKernelGGL(cnn_grad_kernel, dim3((unsigned)blocks), dim3(kCnnThreads), lds, stream, net, samples, n, P,
                           logpsi, O);
        NQS_HIP_TRY(hipGetLastError());
    }
    if (vjp_in) {
        // vjp_out = O^T vjp_in through blocks of rows of O in the workspace
        const int64_t chunk = std::max<int64_t>(1, std::min<int64_t>(n, (int64_t)(256ll << 20) / (P * 4)));
        float *Ow = (float *)workspace(sizeof(float) * (size_t)chunk * P, stream);
        if (!Ow) return set_error(NQS_ENOMEM, "workspace allocation failed");
        for (int64_t k0 = 0; k0 < n; k0 += chunk) {
            const int64_t kn = std::min(chunk, n - k0);
            const int64_t blocks = std::min<int64_t>(kn, (int64_t)device_cus() * 16);
            hipLaunchKernelGGL(cnn_grad_kernel, dim3((unsigned)blocks), dim3(kCnnThreads), lds, stream, net,
                               samples + k0 * S, kn, P, nullptr, Ow);
            st = launch_vjp_chunk(Ow, vjp_in + k0, kn, P, vjp_out, k0 == 0, stream);
            if (st != NQS_OK) return st;
        }
    }
    return NQS_OK;
}

}  // namespace nqs
