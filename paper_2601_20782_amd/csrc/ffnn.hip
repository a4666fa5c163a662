// Dense networks: h_l = ReLU(W_l h_{l-1} + b_l) for l < L, log psi = sum log cosh(z_L).
// This file builds the reduced-precision copies and holds the log-derivative
// (backward) kernel; the MFMA sampler and local energies live in ffnn_mc.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.h"
#include "expand.h"
#include "ffnn_reg.h"
#include "internal.h"

namespace nqs {

// ---------------------------------------------------------------------------
// Copy builder.  For every layer: the format-rounded weights as FP32 values
// in both orientations and FP32 biases.  For the matrix-core path the second
// layer is also kept zero-padded to [ceil(w2/64)*64][ceil(w1/16)*16] (FP32
// values and raw 16-bit codes), and the first layer transposed, [N][w1 pad],
// as raw codes for the LDS-resident rank-1/2 updates.
// ---------------------------------------------------------------------------
__global__ void ffnn_round_layer_kernel(const double *__restrict__ Wsrc, const double *__restrict__ bsrc, int out,
                                        int in, int dtype, float *W, float *Wt, float *b)
{
    const int64_t n = (int64_t)out * in;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n + out; p += (int64_t)gridDim.x * blockDim.x) {
        if (p < n) {
            const int r = (int)(p / in), k = (int)(p % in);
            const float v = (float)round_to_dtype(Wsrc[p], dtype);
            W[p] = v;
            Wt[(int64_t)k * out + r] = v;
        } else {
            b[p - n] = (float)round_to_dtype(bsrc[p - n], dtype);
        }
    }
}

// dst[r][c] (ld_dst, zero padded to rows_p x cols_p) from src[r][c] (ld_src); frag, frag32: the codes, the FP32 values
// in matrix-instruction order (frag_index16, frag_index32) instead of row by row
__global__ void ffnn_pad_kernel(const float *__restrict__ src, int rows, int cols, int ld_src, int rows_p, int cols_p,
                                int dtype, uint16_t *codes, float *f32, int frag, int frag32)
{
    const int64_t n = (int64_t)rows_p * cols_p;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(p / cols_p), c = (int)(p % cols_p);
        const float v = (r < rows && c < cols) ? src[(int64_t)r * ld_src + c] : 0.0f;
        if (f32) f32[frag32 ? frag_index32(r, c, cols_p) : (size_t)p] = v;
        if (codes) {
            uint16_t code;
            if (dtype == kF16) {
                const _Float16 h = (_Float16)v;   // exact: v is an f16 value
                memcpy(&code, &h, 2);
            } else {
                code = (uint16_t)(__float_as_uint(v) >> 16);   // exact: v is a bf16 value
            }
            codes[frag ? frag_index16(r, c, cols_p) : (size_t)p] = code;
        }
    }
}

// ---------------------------------------------------------------------------
// FP8 (E4M3) copy.  Every weight tensor W_l and bias b_l has its own scale
// amax/448 (FP32) and values q * scale, q an E4M3 code (the downcast of the
// two-copy scheme, App. A extended to FP8).  The matrix cores multiply the
// codes: W_l as [Np][Kp] bytes, the layer input as codes of the spins (+-1,
// exact) or of h_{l-1} / s_l, where s_l = 2^ceil(log2(B_l / 448)) and B_l
// bounds |h_l| over every configuration (B_0 = 1, B_l = max_k sum_i
// |W_l[k,i]| B_{l-1} + |b_l[k]| on the rounded values), so no scaled input
// exceeds 448.  The products are accumulated in FP32 and scaled back by
// sW_l s_l.
// ---------------------------------------------------------------------------

// OCP E4M3 code of a value that is exactly representable in the format.
__device__ __forceinline__ uint8_t e4m3_code_exact(double q)
{
    const uint32_t sign = q < 0.0 || (q == 0.0 && signbit(q)) ? 0x80u : 0u;
    const double a = fabs(q);
    if (a == 0.0) return (uint8_t)sign;
    int e;
    const double m = frexp(a, &e);            // a = m 2^e, m in [0.5, 1)
    const int E = e - 1;                      // a = (2m) 2^E, 2m in [1, 2)
    if (E < -6) return (uint8_t)(sign | (uint32_t)(a * 512.0));        // subnormal: a / 2^-9
    return (uint8_t)(sign | ((uint32_t)(E + 7) << 3) | (uint32_t)((2.0 * m - 1.0) * 8.0));
}

// codes of W[out][in] / scale (zero padded to Np x Kp, in matrix-instruction order) and the transposed FP32 values
__global__ void ffnn_e4m3_codes_kernel(const double *__restrict__ W, int out, int in,
                                       const unsigned long long *__restrict__ amax_bits, int Np, int Kp,
                                       uint8_t *__restrict__ codes, float *__restrict__ Wt)
{
    const double amax = __longlong_as_double((long long)*amax_bits);
    const float scale = amax > 0.0 ? (float)(amax / 448.0) : 1.0f;
    const int64_t n = (int64_t)Np * Kp;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(p / Kp), c = (int)(p % Kp);
        uint8_t code = 0;
        if (r < out && c < in) {
            const double q = round_to_dtype(W[(int64_t)r * in + c] / (double)scale, kE4M3);
            code = e4m3_code_exact(q);
            Wt[(int64_t)c * out + r] = (float)(q * (double)scale);
        }
        codes[frag_index8(r, c, Kp)] = code;
    }
}

// Per row k of W (one wave each): rs[k] = sum_i |q_ki| and bq[k] = |q_bk|, with q the E4M3 values
// before scaling (multiples of 2^-9 below 448: the FP64 sums are exact in any order).
__global__ void ffnn_e4m3_rowsum_kernel(const double *__restrict__ W, const double *__restrict__ b, int out, int in,
                                        const unsigned long long *__restrict__ amax_w,
                                        const unsigned long long *__restrict__ amax_b, double *rs, double *bq)
{
    const int r = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= out) return;
    const double aw = __longlong_as_double((long long)*amax_w), ab = __longlong_as_double((long long)*amax_b);
    const float sw = aw > 0.0 ? (float)(aw / 448.0) : 1.0f, sb = ab > 0.0 ? (float)(ab / 448.0) : 1.0f;
    double acc = 0.0;
    for (int c = lane; c < in; c += 64) acc += fabs(round_to_dtype(W[(int64_t)r * in + c] / (double)sw, kE4M3));
    acc = group_sum<64>(acc);
    if (lane == 0) {
        rs[r] = acc;
        bq[r] = fabs(round_to_dtype(b[r] / (double)sb, kE4M3));
    }
}

static nqs_status ffnn_build_e4m3(nqs_model *m, hipStream_t stream)
{
    const nqs_model_desc &d = m->desc;
    Copy &c = m->copies[NQS_FP8_E4M3];
    FfnnDev &f = c.ffnn;
    const int L = d.n_layers;
    f.n_layers = L;
    f.widths[0] = d.n_visible;
    for (int l = 0; l < L; ++l) f.widths[l + 1] = d.widths[l];
    f.m1p = f.m2p = 0;   // the two-layer register kernels take 16-bit copies only
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    size_t bytes = al(sizeof(unsigned long long) * 2 * L);
    for (int l = 0; l < L; ++l) {
        const size_t n = (size_t)f.widths[l + 1] * f.widths[l];
        f.Kp[l] = (f.widths[l] + 127) / 128 * 128;   // 128 one-byte codes per contraction step
        f.Np[l] = (f.widths[l + 1] + 127) / 128 * 128;
        bytes += 2 * al(sizeof(float) * n) + al(sizeof(float) * f.widths[l + 1]) + al((size_t)f.Np[l] * f.Kp[l]) +
                 al(sizeof(float) * f.Np[l]) + 2 * al(sizeof(double) * f.widths[l + 1]);
    }
    if (!c.block) NQS_HIP_TRY(hipMalloc(&c.block, bytes));
    char *base = (char *)c.block;
    auto carve = [&](size_t sz) {
        char *p = base;
        base += al(sz);
        return p;
    };
    unsigned long long *amax = (unsigned long long *)carve(sizeof(unsigned long long) * 2 * L);
    double *rs[NQS_MAX_LAYERS], *bq[NQS_MAX_LAYERS];
    int64_t off = 0;
    for (int l = 0; l < L; ++l) {
        const int out = f.widths[l + 1], in = f.widths[l];
        const int64_t n = (int64_t)out * in;
        f.W[l] = (float *)carve(sizeof(float) * n);
        f.Wt[l] = (float *)carve(sizeof(float) * n);
        f.b[l] = (float *)carve(sizeof(float) * out);
        f.Wd[l] = carve((size_t)f.Np[l] * f.Kp[l]);
        f.bd[l] = (float *)carve(sizeof(float) * f.Np[l]);
        rs[l] = (double *)carve(sizeof(double) * out);
        bq[l] = (double *)carve(sizeof(double) * out);
        const double *Wm = m->master + off, *bm = m->master + off + n;
        nqs_status e = launch_e4m3_tensor(Wm, n, amax + 2 * l, f.W[l], stream);
        if (e != NQS_OK) return e;
        e = launch_e4m3_tensor(bm, out, amax + 2 * l + 1, f.b[l], stream);
        if (e != NQS_OK) return e;
        const int64_t nc = (int64_t)f.Np[l] * f.Kp[l];
        hipLaunchKernelGGL(ffnn_e4m3_codes_kernel, dim3((unsigned)std::min<int64_t>((nc + 255) / 256, 8192)), dim3(256),
                           0, stream, Wm, out, in, (const unsigned long long *)(amax + 2 * l), f.Np[l], f.Kp[l],
                           (uint8_t *)f.Wd[l], f.Wt[l]);
        hipLaunchKernelGGL(ffnn_pad_kernel, dim3((f.Np[l] + 255) / 256), dim3(256), 0, stream, f.b[l], 1, out, out, 1,
                           f.Np[l], (int)kF32, (uint16_t *)nullptr, f.bd[l], 0, 0);
        hipLaunchKernelGGL(ffnn_e4m3_rowsum_kernel, dim3((out + 3) / 4), dim3(256), 0, stream, Wm, bm, out, in,
                           (const unsigned long long *)(amax + 2 * l), (const unsigned long long *)(amax + 2 * l + 1),
                           rs[l], bq[l]);
        NQS_HIP_TRY(hipGetLastError());
        off += n + out;
    }
    if ((size_t)(base - (char *)c.block) > bytes) return set_error(NQS_EDEVICE, "internal layout overflow");
    // scales on the host: weight scales from the amax words, input scales from the bounds B_l
    std::vector<unsigned long long> hmax(2 * L);
    NQS_HIP_TRY(hipMemcpyAsync(hmax.data(), amax, sizeof(unsigned long long) * 2 * L, hipMemcpyDeviceToHost, stream));
    std::vector<std::vector<double>> hrs(L), hbq(L);
    for (int l = 0; l + 1 < L; ++l) {
        hrs[l].resize(f.widths[l + 1]);
        hbq[l].resize(f.widths[l + 1]);
        NQS_HIP_TRY(hipMemcpyAsync(hrs[l].data(), rs[l], sizeof(double) * f.widths[l + 1], hipMemcpyDeviceToHost, stream));
        NQS_HIP_TRY(hipMemcpyAsync(hbq[l].data(), bq[l], sizeof(double) * f.widths[l + 1], hipMemcpyDeviceToHost, stream));
    }
    NQS_HIP_TRY(hipStreamSynchronize(stream));
    auto scale_of = [](unsigned long long bits) {
        double a;
        std::memcpy(&a, &bits, sizeof(double));
        return a > 0.0 ? (float)(a / 448.0) : 1.0f;
    };
    double B = 1.0;          // bound on |input of layer l| (spins)
    float s_in = 1.0f;       // scale of the input of layer l
    for (int l = 0; l < L; ++l) {
        const float sw = scale_of(hmax[2 * l]), sb = scale_of(hmax[2 * l + 1]);
        f.acc_scale[l] = sw * s_in;   // s_in is a power of two: exact
        if (l + 1 < L) {
            double Bn = 0.0;
            for (int k = 0; k < f.widths[l + 1]; ++k)
                Bn = std::max(Bn, ((double)sw * hrs[l][k]) * B + (double)sb * hbq[l][k]);
            const float s_next = Bn > 0.0 ? (float)std::ldexp(1.0, (int)std::ceil(std::log2(Bn / 448.0))) : 1.0f;
            f.next_inv[l] = 1.0f / s_next;   // exact: a power of two
            B = Bn;
            s_in = s_next;
        } else {
            f.next_inv[l] = 1.0f;
        }
    }
    c.valid = true;
    return NQS_OK;
}

nqs_status ffnn_build_copy(nqs_model *m, int dtype, hipStream_t stream)
{
    const nqs_model_desc &d = m->desc;
    if (dtype == NQS_FP8_E4M3) return ffnn_build_e4m3(m, stream);
    Copy &c = m->copies[dtype];
    FfnnDev &f = c.ffnn;
    f.n_layers = d.n_layers;
    f.widths[0] = d.n_visible;
    for (int l = 0; l < d.n_layers; ++l) f.widths[l + 1] = d.widths[l];
    const bool lp = dtype == NQS_BF16 || dtype == NQS_F16;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const int N = f.widths[0], M1 = f.widths[1];
    f.m1p = (M1 + 63) / 64 * 64;   // lane k of a wave owns hidden units k + 64 q
    f.m2p = f.n_layers >= 2 ? (f.widths[2] + 63) / 64 * 64 : 0;
    size_t bytes = 0;
    for (int l = 0; l < f.n_layers; ++l) {
        const size_t n = (size_t)f.widths[l + 1] * f.widths[l];
        bytes += 2 * al(sizeof(float) * n) + al(sizeof(float) * f.widths[l + 1]);
    }
    if (f.n_layers >= 2)
        bytes += al(sizeof(uint16_t) * (size_t)f.m2p * f.m1p) + al(sizeof(uint16_t) * (size_t)N * f.m1p) +
                 al(sizeof(float) * (size_t)f.m2p * f.m1p) + al(sizeof(float) * (size_t)N * f.m1p) +
                 al(sizeof(float) * f.m1p) + al(sizeof(float) * f.m2p);
    const size_t esize = lp ? sizeof(uint16_t) : sizeof(float);
    for (int l = 0; l < f.n_layers; ++l) {
        f.Kp[l] = (f.widths[l] + 63) / 64 * 64;
        f.Np[l] = (f.widths[l + 1] + 127) / 128 * 128;
        bytes += al(esize * (size_t)f.Np[l] * f.Kp[l]) + al(sizeof(float) * f.Np[l]);
    }
    if (!c.block) NQS_HIP_TRY(hipMalloc(&c.block, bytes));
    char *base = (char *)c.block;
    auto carve = [&](size_t sz) {
        char *p = base;
        base += al(sz);
        return p;
    };
    for (int l = 0; l < f.n_layers; ++l) {
        const size_t n = (size_t)f.widths[l + 1] * f.widths[l];
        f.W[l] = (float *)carve(sizeof(float) * n);
        f.Wt[l] = (float *)carve(sizeof(float) * n);
        f.b[l] = (float *)carve(sizeof(float) * f.widths[l + 1]);
    }
    int64_t off = 0;
    for (int l = 0; l < f.n_layers; ++l) {
        const int out = f.widths[l + 1], in = f.widths[l];
        const int64_t n = (int64_t)out * in;
        const int blocks = (int)std::min<int64_t>((n + out + 255) / 256, 8192);
        hipLaunchKernelGGL(ffnn_round_layer_kernel, dim3(blocks), dim3(256), 0, stream, m->master + off,
                           m->master + off + n, out, in, dtype, f.W[l], f.Wt[l], f.b[l]);
        NQS_HIP_TRY(hipGetLastError());
        off += n + out;
    }
    if (f.n_layers >= 2) {
        const int M2 = f.widths[2];
        f.W2c = (uint16_t *)carve(sizeof(uint16_t) * (size_t)f.m2p * f.m1p);
        f.W1ct = (uint16_t *)carve(sizeof(uint16_t) * (size_t)N * f.m1p);
        f.W2p = (float *)carve(sizeof(float) * (size_t)f.m2p * f.m1p);
        f.W1tp = (float *)carve(sizeof(float) * (size_t)N * f.m1p);
        f.b1p = (float *)carve(sizeof(float) * f.m1p);
        f.b2p = (float *)carve(sizeof(float) * f.m2p);
        auto pad = [&](const float *src, int rows, int cols, int ld, int rows_p, int cols_p, uint16_t *codes, float *f32,
                       int frag32 = 0) {
            const int64_t n = (int64_t)rows_p * cols_p;
            const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
            hipLaunchKernelGGL(ffnn_pad_kernel, dim3(blocks), dim3(256), 0, stream, src, rows, cols, ld, rows_p, cols_p,
                               dtype, codes, f32, 0, frag32);
        };
        pad(f.W[1], M2, M1, M1, f.m2p, f.m1p, lp ? f.W2c : nullptr, lp ? nullptr : f.W2p, 1);
        pad(f.Wt[0], N, M1, M1, N, f.m1p, lp ? f.W1ct : nullptr, f.W1tp);
        pad(f.b[0], 1, M1, M1, 1, f.m1p, nullptr, f.b1p);
        pad(f.b[1], 1, M2, M2, 1, f.m2p, nullptr, f.b2p);
        NQS_HIP_TRY(hipGetLastError());
    }
    for (int l = 0; l < f.n_layers; ++l) {
        const int out = f.widths[l + 1], in = f.widths[l];
        f.Wd[l] = carve(esize * (size_t)f.Np[l] * f.Kp[l]);
        f.bd[l] = (float *)carve(sizeof(float) * f.Np[l]);
        const int64_t n = (int64_t)f.Np[l] * f.Kp[l];
        const int blocks = (int)std::min<int64_t>((n + 255) / 256, 8192);
        hipLaunchKernelGGL(ffnn_pad_kernel, dim3(blocks), dim3(256), 0, stream, f.W[l], out, in, in, f.Np[l], f.Kp[l],
                           dtype, lp ? (uint16_t *)f.Wd[l] : nullptr, lp ? nullptr : (float *)f.Wd[l], 1, 0);
        hipLaunchKernelGGL(ffnn_pad_kernel, dim3((f.Np[l] + 255) / 256), dim3(256), 0, stream, f.b[l], 1, out, out, 1,
                           f.Np[l], dtype, (uint16_t *)nullptr, f.bd[l], 0, 0);
        NQS_HIP_TRY(hipGetLastError());
    }
    NQS_HIP_TRY(hipStreamSynchronize(stream));
    c.valid = true;
    return NQS_OK;
}

// ---------------------------------------------------------------------------
// log psi and O_k by reverse-mode differentiation written out by hand.
// One block per sample (grid-stride); activations stay in LDS.
//   delta_L = tanh(z_L);  O_{b_l} = delta_l;  O_{W_l} = delta_l (x) h_{l-1};
//   delta_{l-1} = (W_l^T delta_l) * [z_{l-1} > 0]   (ReLU'(0) = 0).
// O rows are written with consecutive threads on consecutive parameters.
// ---------------------------------------------------------------------------
struct GradArgs {
    FfnnDev net;
    const int8_t *samples;
    int64_t n;
    float *logpsi;
    float *O;         // columns [p0, p1) of O, row stride p1 - p0
    int64_t P;
    int64_t p0, p1;
    int lds_stride;   // floats reserved per layer activation vector
};

__global__ void __launch_bounds__(256) ffnn_grad_kernel(GradArgs A)
{
    extern __shared__ float smem[];
    const FfnnDev &net = A.net;
    const int L = net.n_layers, N = net.widths[0];
    const int S = A.lds_stride;
    float *in0 = smem;                  // [N] spins
    float *z = smem + S;                // [L][S] pre-activations
    float *dl = z + (size_t)L * S;      // [2][S] deltas (ping-pong)
    __shared__ float red[4];
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int64_t smp = blockIdx.x; smp < A.n; smp += gridDim.x) {
        for (int i = tid; i < N; i += nt) in0[i] = (float)A.samples[smp * N + i];
        __syncthreads();
        // forward
        for (int l = 0; l < L; ++l) {
            const int out = net.widths[l + 1], in = net.widths[l];
            const float *src = l == 0 ? in0 : z + (size_t)(l - 1) * S;
            const float *Wt = net.Wt[l];
            for (int r = tid; r < out; r += nt) {
                float acc = net.b[l][r];
                if (l == 0) {
                    for (int k = 0; k < in; ++k) acc = fmaf(Wt[(size_t)k * out + r], src[k], acc);
                } else {
                    for (int k = 0; k < in; ++k) acc = fmaf(Wt[(size_t)k * out + r], fmaxf(src[k], 0.0f), acc);
                }
                z[(size_t)l * S + r] = acc;
            }
            __syncthreads();
        }
        // log psi
        const int wl = net.widths[L];
        float part = 0.0f;
        for (int r = tid; r < wl; r += nt) part += logcosh_f32(z[(size_t)(L - 1) * S + r]);
        part = group_sum<64>(part);
        if ((tid & 63) == 0) red[tid >> 6] = part;
        __syncthreads();
        if (tid == 0 && A.logpsi) A.logpsi[smp] = red[0] + red[1] + red[2] + red[3];
        if (A.O) {
            const int64_t p0 = A.p0, p1 = A.p1;
            float *O = A.O + smp * (p1 - p0) - p0;   // O[p] for p in [p0, p1)
            // parameter offsets
            int64_t offW[NQS_MAX_LAYERS], offb[NQS_MAX_LAYERS], off = 0;
            for (int l = 0; l < L; ++l) {
                offW[l] = off;
                off += (int64_t)net.widths[l + 1] * net.widths[l];
                offb[l] = off;
                off += net.widths[l + 1];
            }
            float *d = dl;
            for (int r = tid; r < wl; r += nt) d[r] = tanhf(z[(size_t)(L - 1) * S + r]);
            __syncthreads();
            for (int l = L - 1; l >= 0; --l) {
                const int out = net.widths[l + 1], in = net.widths[l];
                const float *src = l == 0 ? in0 : z + (size_t)(l - 1) * S;
                for (int r = tid; r < out; r += nt)
                    if (offb[l] + r >= p0 && offb[l] + r < p1) O[offb[l] + r] = d[r];
                // O_W[r][k] = d[r] * h[k], consecutive threads on consecutive k; rows
                // [r0, r1) of this layer meet the column range
                const int r0 = (int)min((int64_t)out, max((int64_t)0, (p0 - offW[l]) / in));
                const int r1 = (int)min((int64_t)out, max((int64_t)0, (p1 - offW[l] + in - 1) / in));
                for (int r = r0; r < r1; ++r) {
                    const float dr = d[r];
                    const int64_t rb = offW[l] + (int64_t)r * in;
                    const int k0 = (int)max((int64_t)0, p0 - rb), k1 = (int)min((int64_t)in, p1 - rb);
                    float *orow = O + rb;
                    if (l == 0) {
                        for (int k = k0 + tid; k < k1; k += nt) orow[k] = dr * src[k];
                    } else {
                        for (int k = k0 + tid; k < k1; k += nt) orow[k] = dr * fmaxf(src[k], 0.0f);
                    }
                }
                // parameters of the layers below lie before offW[l]
                if (l == 0 || offW[l] <= p0) break;
                float *dn = (d == dl) ? dl + S : dl;
                const float *W = net.W[l];
                for (int k = tid; k < in; k += nt) {
                    float g = 0.0f;
                    for (int r = 0; r < out; ++r) g = fmaf(W[(size_t)r * in + k], d[r], g);
                    dn[k] = src[k] > 0.0f ? g : 0.0f;
                }
                __syncthreads();
                d = dn;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Factors of O for many samples: the layer inputs a_{l-1} and the deltas of every layer, whose outer products are
// the blocks of O.  Forward and backward pass are products of the samples' rows with the layer's weights on the
// FP32 matrix cores:
//   z_l = a_{l-1} W_l^T + b_l (k in order, starting at the bias),  delta_{l-1} = (delta_l W_l) * [a_{l-1} > 0].
// v_mfma_f32_16x16x4_f32 adds its four products one after another with one rounding each, so every sum is the
// chain of fmaf of ffnn_grad_kernel (one block per sample) and the factors reproduce its O bit for bit.  No split of
// the contraction: it would change the chain.
//
// 64 samples x 64 outputs per block of four waves (2 x 2 tiles of 16 x 16 each), 32 contraction steps per barrier,
// the next ones loaded into registers meanwhile; row strides of 36 and 80 floats spread a fragment read over all 64
// banks.  log psi of 4096 samples of the 100-400-200 network: 48 us (five
// launches; the products take half of it) against 175 us with one block per sample, whose sums wait for L2.
// ---------------------------------------------------------------------------
constexpr int kGmTile = 64, kGmStep = 32, kGmLdx = 36, kGmLdb = 80;
constexpr int64_t kFactorSamples = 65535 * (int64_t)kGmTile;   // of one launch (tiles of samples along the grid's y)
typedef float gm_f32x4 __attribute__((ext_vector_type(4)));

struct FactorGemmArgs {
    const float *X;      // [n][ldx], K columns
    const float *B;      // [K][N]
    const float *bias;   // [N] start of the sums, or NULL (0)
    const float *mask;   // [n][ldm]: outputs where it is not positive are 0; or NULL
    float *out;          // [n][ldo], N columns
    int64_t n, ldx, ldm, ldo;
    int K, N, relu;
};

__global__ void __launch_bounds__(256) ffnn_factor_gemm_kernel(FactorGemmArgs A)
{
    __shared__ float Xs[2][kGmTile * kGmLdx], Bs[2][kGmStep * kGmLdb];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, la = lane & 15, lk = lane >> 4;
    const int64_t m0 = blockIdx.y * (int64_t)kGmTile;
    const int n0 = blockIdx.x * kGmTile, wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    // staging: rows xr + 8 i of X at step xk; steps br + 4 i of B at column bc
    const int xk = tid & 31, xr = tid >> 5, bc = tid & 63, br = tid >> 6;
    float xv[8], bv[8];
    auto load = [&](int k0) {
        // every load is made, from a valid place (a branch around a load waits for all loads in flight); rows and
        // columns past the last feed outputs that are not stored
        const int k = k0 + xk;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float x = A.X[min(m0 + xr + 8 * i, A.n - 1) * A.ldx + min(k, A.K - 1)];
            const int kb = k0 + br + 4 * i;
            const float b = A.B[(size_t)min(kb, A.K - 1) * A.N + min(n0 + bc, A.N - 1)];
            xv[i] = k < A.K ? x : 0.0f;
            bv[i] = kb < A.K ? b : 0.0f;
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            Xs[buf][(xr + 8 * i) * kGmLdx + xk] = xv[i];
            Bs[buf][(br + 4 * i) * kGmLdb + bc] = bv[i];
        }
    };
    gm_f32x4 acc[2][2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int col = n0 + wn + 16 * b + la;
        const float v = A.bias && col < A.N ? A.bias[col] : 0.0f;
#pragma unroll
        for (int a = 0; a < 2; ++a) acc[a][b] = gm_f32x4{v, v, v, v};
    }
    load(0);
    store(0);
    int buf = 0;
    for (int k0 = 0; k0 < A.K; k0 += kGmStep) {
        __syncthreads();
        const bool more = k0 + kGmStep < A.K;
        if (more) load(k0 + kGmStep);
#pragma unroll
        for (int s = 0; s < kGmStep / 4; ++s) {
            float a[2], b[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                a[q] = Xs[buf][(wm + 16 * q + la) * kGmLdx + 4 * s + lk];
                b[q] = Bs[buf][(4 * s + lk) * kGmLdb + wn + 16 * q + la];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (more) store(buf ^ 1);
        buf ^= 1;
    }
    // D[i][j] of a 16 x 16 block: j = lane % 16 (output), i = 4 (lane / 16) + register (sample)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t row = m0 + wm + 16 * i + 4 * lk + r;
                const int col = n0 + wn + 16 * j + la;
                if (row >= A.n || col >= A.N) continue;
                float v = acc[i][j][r];
                if (A.relu) v = fmaxf(v, 0.0f);
                if (A.mask) v = A.mask[row * A.ldm + col] > 0.0f ? v : 0.0f;
                A.out[row * A.ldo + col] = v;
            }
}

// spins as the first layer's inputs (row stride sa)
__global__ void ffnn_factor_spins_kernel(const int8_t *__restrict__ samples, int64_t n, int N, int64_t sa,
                                         float *__restrict__ acts)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= n * N) return;
    const int64_t k = e / N;
    acts[k * sa + (e - k * N)] = (float)samples[e];
}

// The head of one sample per block: log psi = sum log cosh z in ffnn_grad_kernel's order, and z -> tanh z in place.
__global__ void __launch_bounds__(256) ffnn_factor_head_kernel(float *z, int64_t n, int64_t ld, int w,
                                                               float *__restrict__ logpsi)
{
    __shared__ float red[4];
    for (int64_t k = blockIdx.x; k < n; k += gridDim.x) {
        float *zk = z + k * ld;
        float part = 0.0f;
        for (int r = threadIdx.x; r < w; r += 256) {
            const float v = zk[r];
            if (logpsi) part += logcosh_f32(v);
            zk[r] = tanhf(v);
        }
        if (!logpsi) continue;
        part = group_sum<64>(part);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
        __syncthreads();
        if (threadIdx.x == 0) logpsi[k] = red[0] + red[1] + red[2] + red[3];
        __syncthreads();
    }
}

// acts [n][sum of the layers' inputs], dels [n][sum of their outputs]; logpsi may be NULL.  Without `backward` only
// the last layer's deltas are formed.
static nqs_status factors_from(const FfnnDev &net, const int8_t *samples, int64_t n, float *acts, float *dels,
                               float *logpsi, bool backward, hipStream_t stream)
{
    const int L = net.n_layers, N = net.widths[0];
    int64_t sa = 0, sd = 0, oa[NQS_MAX_LAYERS], od[NQS_MAX_LAYERS];
    for (int l = 0; l < L; ++l) {
        oa[l] = sa;
        od[l] = sd;
        sa += net.widths[l];
        sd += net.widths[l + 1];
    }
    const int64_t sb = (n * N + 255) / 256, my = (n + kGmTile - 1) / kGmTile;
    if (n > kFactorSamples) return set_error(NQS_EINVAL, "too many samples");
    hipLaunchKernelGGL(ffnn_factor_spins_kernel, dim3((unsigned)sb), dim3(256), 0, stream, samples, n, N, sa, acts);
    auto gemm = [&](const FactorGemmArgs &G) {
        hipLaunchKernelGGL(ffnn_factor_gemm_kernel, dim3((unsigned)((G.N + kGmTile - 1) / kGmTile), (unsigned)my),
                           dim3(256), 0, stream, G);
    };
    for (int l = 0; l < L; ++l) {
        const bool last = l + 1 == L;
        gemm(FactorGemmArgs{acts + oa[l], net.Wt[l], net.b[l], nullptr, last ? dels + od[l] : acts + oa[l + 1], n, sa, 0,
                            last ? sd : sa, net.widths[l], net.widths[l + 1], last ? 0 : 1});
    }
    hipLaunchKernelGGL(ffnn_factor_head_kernel, dim3((unsigned)std::min<int64_t>(n, 65536)), dim3(256), 0, stream,
                       dels + od[L - 1], n, sd, net.widths[L], logpsi);
    for (int l = L - 1; backward && l >= 1; --l)
        gemm(FactorGemmArgs{dels + od[l], net.W[l], nullptr, acts + oa[l], dels + od[l - 1], n, sd, sa, sd,
                            net.widths[l + 1], net.widths[l], 0});
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

// O [n][p1 - p0] from the factors: one multiply per value, bound by the writes.  A block writes kExpandSpan
// consecutive parameters of one sample, so its stores run through memory in order, from the factors that these meet in
// LDS (all of a sample's would not fit it for every network that the gradient takes: 165 KB for eight layers of 2,752
// units); 16 bytes a store where every layer's rows and O's are multiples of 16 bytes.  4096 samples of the 100-400-200
// network (1.98 GB): 482 us with the factors, 4.5 TB/s for this kernel (a copy reaches 5.2, read and written);
// 905 us when a block wrote 4 KB of each of 16 samples, 1762 us with one block per sample for everything.
// Small networks of several blocks a sample keep all deltas and inputs of the layers met (WHOLE): 4001 samples of
// 100-400-200 take 451 us wherever O lies, 452 to 473 with only the needed ones; beyond 10 KB of factors these are as
// fast or faster (64-2048-2048-2048, 100 samples: 1,063 us against 1,365).
// V consecutive parameters per thread and store (1, or 4 where every row is a multiple of 4 floats)
// WHOLE: all deltas and inputs of the layers that the span meets, else only those that it needs
template <int V, bool WHOLE>
__global__ void __launch_bounds__(256) ffnn_expand_kernel(ExpandArgs E, int spans)
{
    extern __shared__ __align__(16) float fac[];   // of each layer that the span meets: inputs, rows' deltas, biases' deltas
    const int64_t k = blockIdx.x / spans;
    const int tid = threadIdx.x;
    const int64_t b0 = E.p0 + (int64_t)(blockIdx.x - k * spans) * kExpandSpan, b1 = min(E.p1, b0 + kExpandSpan);
    float *f = fac;
    for (int l = 0; l < E.L; ++l) {
        const ExpandPart x = expand_part(E, l, b0, b1);
        const float *d = E.dels + k * E.sd + E.offD[l];
        if (WHOLE ? x.rows + x.nd > 0 : x.rows > 0) {
            const int in = E.in[l], r0 = WHOLE ? 0 : (int)x.r0, rows = WHOLE ? E.out[l] : x.rows;
            for (int i = tid; i < rows; i += 256) f[((in + 3) & ~3) + i] = d[r0 + i];
            for (int i = tid; i < in; i += 256) f[i] = E.acts[k * E.sa + E.offA[l] + i];
            f += expand_words(in, rows, 0);
        }
        if (WHOLE) continue;
        for (int i = tid; i < x.nd; i += 256) f[i] = d[x.d0 + i];
        f += (x.nd + 3) & ~3;
    }
    __syncthreads();
    float *O = E.O + k * (E.p1 - E.p0) + (b0 - E.p0);
    f = fac;
    for (int l = 0; l < E.L; ++l) {
        const ExpandPart x = expand_part(E, l, b0, b1);
        const unsigned in = (unsigned)E.in[l], inv = E.inv[l];
        const float *a = f, *d = f + ((in + 3) & ~3u);   // the deltas from the first row met on
        if (WHOLE) {
            if (x.rows + x.nd > 0) f += expand_words((int)in, E.out[l], 0);
        } else {
            f += expand_words((int)in, x.rows, 0);
        }
        if (x.rows > 0) {
            if (WHOLE) d += x.r0;
            // position q0 + t is row r0 + r, column c; t advanced by 256 V with (r, c) carried
            const unsigned c0 = x.q0 - x.r0 * in + tid * V;
            unsigned r = expand_div(c0, in, inv), c = c0 - r * in;
            const unsigned dr = expand_div(256 * V, in, inv), dc = 256 * V - dr * in;
            for (unsigned t = tid * V; t < x.count; t += 256 * V) {
                const float dv = d[r];
                if constexpr (V == 4) {
                    const float4 av = *reinterpret_cast<const float4 *>(a + c);
                    *reinterpret_cast<float4 *>(O + t) = make_float4(dv * av.x, dv * av.y, dv * av.z, dv * av.w);
                } else {
                    O[t] = dv * a[c];
                }
                r += dr;
                c += dc;
                if (c >= in) {
                    c -= in;
                    ++r;
                }
            }
            O += x.count;
        }
        const float *b = WHOLE ? a + ((in + 3) & ~3u) + x.d0 : f;
        for (int i = tid; i < x.nd; i += 256) O[i] = b[i];
        if (!WHOLE) f += (x.nd + 3) & ~3;
        O += x.nd;
    }
}

static ExpandArgs expand_args(const FfnnDev &net)
{
    ExpandArgs E{};
    E.L = net.n_layers;
    int64_t off = 0;
    for (int l = 0; l < E.L; ++l) {
        E.in[l] = net.widths[l];
        E.out[l] = net.widths[l + 1];
        E.inv[l] = 0xFFFFFFFFu / (unsigned)net.widths[l];
        E.offW[l] = off;
        E.offA[l] = E.sa;
        E.offD[l] = E.sd;
        off += (int64_t)E.out[l] * E.in[l] + E.out[l];
        E.sa += E.in[l];
        E.sd += E.out[l];
    }
    E.offW[E.L] = off;
    return E;
}

// columns [p0, p1) of O of the n samples whose factors E holds
static nqs_status expand_columns(ExpandArgs E, int64_t n, int64_t p0, int64_t p1, float *O, hipStream_t stream)
{
    E.n = n;
    E.p0 = p0;
    E.p1 = p1;
    bool vec = (p1 - p0) % 4 == 0 && p0 % 4 == 0 && (uintptr_t)O % 16 == 0;
    for (int l = 0; l < E.L; ++l) vec = vec && E.in[l] % 4 == 0 && E.out[l] % 4 == 0;
    const int64_t spans = (p1 - p0 + kExpandSpan - 1) / kExpandSpan;
    const int64_t most = (((int64_t)1 << 24) - 1) / spans;   // samples per launch: fewer than 2^32 threads
    int all = 0;
    for (int l = 0; l < E.L; ++l) all += expand_words(E.in[l], E.out[l], 0);
    const bool whole = vec && spans > 1 && all <= 2560;
    const size_t lds = sizeof(float) * (size_t)(whole ? all : expand_lds_words(E));
    for (int64_t k0 = 0; k0 < n; k0 += most) {
        ExpandArgs C = E;
        C.n = std::min(most, n - k0);
        C.acts += k0 * E.sa;
        C.dels += k0 * E.sd;
        C.O = O + k0 * (p1 - p0);
        auto launch = [&](auto kernel) {
            allow_lds(kernel, lds);
            hipLaunchKernelGGL(kernel, dim3((unsigned)(C.n * spans)), dim3(256), lds, stream, C, (int)spans);
        };
        if (whole) launch(ffnn_expand_kernel<4, true>);
        else if (vec) launch(ffnn_expand_kernel<4, false>);
        else launch(ffnn_expand_kernel<1, false>);
    }
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

nqs_status ffnn_logpsi_grad(nqs_model *m, const int8_t *samples, int64_t n, float *logpsi, float *O,
                            const float *vjp_in, float *vjp_out, hipStream_t stream, int64_t p0, int64_t p1)
{
    nqs_status st = ensure_copy(m, NQS_F32, stream);
    if (st != NQS_OK) return st;
    const FfnnDev &net = m->copies[NQS_F32].ffnn;
    int maxw = net.widths[0];
    for (int l = 1; l <= net.n_layers; ++l) maxw = std::max(maxw, net.widths[l]);
    GradArgs A;
    A.net = net;
    A.P = m->P;
    A.p0 = p0;
    A.p1 = p1;
    A.lds_stride = (maxw + 3) & ~3;
    const size_t lds = sizeof(float) * (size_t)A.lds_stride * (1 + net.n_layers + 2);
    if (lds > 160 * 1024) return set_error(NQS_EUNSUPPORTED, "network too wide for the gradient kernel");
    allow_lds(ffnn_grad_kernel, lds);
    // Small calls, and calls under capture or without scratch, take one block per sample; the others form the factors
    // and expand them, chunk by chunk.  The values are the same bit for bit.  The line: 16-64-32, 512 samples 36 us as one
    // block per sample (its chains' latency; 126 us at 4096 samples against 43), 36-144-72, 64 samples 68 against 39;
    // log psi alone 36-144-72, 1024 samples 21 against 28 (five launches), 64-256-128 34 against 29.  Some columns: while
    // the samples' blocks run all at once and write little, 513 samples of 36-144-72, 317 columns 45 against 51, of
    // 25-100-50, 1,912 columns 41 against 47 (4,096 samples: 94 against 61).
    const double P = (double)m->P, nP = (double)n * P, w = (double)(p1 - p0);
    const bool small = !O                ? P < 3.0e4 && nP < 3.0e7
                       : p1 - p0 == m->P ? P < 1.2e4 && nP < 2.5e6
                                         : n <= 2048 && n * w < 2.5e6 && (P < 1.2e4 || (P < 2.0e4 && 16 * w <= P));
    bool todo = logpsi || O;
    if (todo && !small && !stream_capturing(stream)) {
        const ScratchLease lease(stream);
        if (float *acts = (float *)lease.ptr()) {
            ExpandArgs E = expand_args(net);
            const int64_t per = E.sa + E.sd;
            const int64_t chunk = std::min({n, (int64_t)(kScratchBytes / sizeof(float)) / per, kFactorSamples});
            float *dels = acts + chunk * E.sa;
            E.acts = acts;
            E.dels = dels;
            for (int64_t k0 = 0; k0 < n; k0 += chunk) {
                const int64_t kn = std::min(chunk, n - k0);
                st = factors_from(net, samples + k0 * net.widths[0], kn, acts, dels, logpsi ? logpsi + k0 : nullptr,
                                  O != nullptr, stream);
                if (st == NQS_OK && O) st = expand_columns(E, kn, p0, p1, O + k0 * (p1 - p0), stream);
                if (st != NQS_OK) return st;
            }
            todo = false;
        }
    }
    if (todo) {
        A.samples = samples;
        A.n = n;
        A.logpsi = logpsi;
        A.O = O;
        hipLaunchKernelGGL(ffnn_grad_kernel, dim3((unsigned)std::min<int64_t>(n, 4096)), dim3(256), lds, stream, A);
        NQS_HIP_TRY(hipGetLastError());
    }
    if (vjp_in) {
        // sum_k g_k delta_k (x) a_k per layer on the FP64 matrix cores, from the factors of up to 256 MiB of samples
        // at a time (100-400-200, 6000 samples: 0.18 ms, half of it the products, against 6.7 ms through blocks of O)
        ExpandArgs E = expand_args(net);
        const int64_t per = E.sa + E.sd;
        const int64_t chunk = std::max<int64_t>(1, std::min({n, ((int64_t)64 << 20) / per, kFactorSamples}));
        FacLayerDesc lay[NQS_MAX_LAYERS];
        for (int l = 0; l < E.L; ++l) lay[l] = FacLayerDesc{nullptr, nullptr, E.sd, E.sa, E.out[l], E.in[l], 0, nullptr};
        const size_t fb = (sizeof(float) * (size_t)(chunk * per) + 255) & ~(size_t)255;
        char *ws = (char *)workspace(fb + fac_vjp_bytes(lay, E.L, chunk), stream);
        if (!ws) return set_error(NQS_ENOMEM, "workspace allocation failed");
        float *acts = (float *)ws, *dels = acts + chunk * E.sa;
        for (int l = 0; l < E.L; ++l) {
            lay[l].U = dels + E.offD[l];
            lay[l].V = acts + E.offA[l];
        }
        for (int64_t k0 = 0; k0 < n; k0 += chunk) {
            const int64_t kn = std::min(chunk, n - k0);
            st = factors_from(net, samples + k0 * net.widths[0], kn, acts, dels, nullptr, true, stream);
            if (st == NQS_OK)
                st = launch_fac_vjp(lay, E.L, kn, chunk, vjp_in + k0, k0 > 0, k0 + kn == n ? vjp_out : nullptr, ws + fb,
                                    stream);
            if (st != NQS_OK) return st;
        }
    }
    return NQS_OK;
}

}  // namespace nqs

namespace nqs {

nqs_status ffnn_sample_dispatch(int dtype, int QK, bool trace, const FfnnSampleArgs &A, int blocks, size_t lds,
                                hipStream_t s);
nqs_status ffnn_eloc_dispatch(int dtype, int QK, const FfnnElocArgs &A, int blocks, size_t lds, hipStream_t s);
bool ffnn_reg_sample_launch_bf16(int ke, bool trace, bool perchain, const FfnnSampleArgs &A, int blocks, size_t lds,
                              hipStream_t s);
bool ffnn_reg_sample_launch_f16(int ke, bool trace, bool perchain, const FfnnSampleArgs &A, int blocks, size_t lds,
                              hipStream_t s);
size_t ffnn_reg_sample_lds_bf16(int N, int ke, int m2p);
size_t ffnn_reg_sample_lds_f16(int N, int ke, int m2p);
bool ffnn_reg_eloc_launch_bf16(int ke, const FfnnElocArgs &A, int G, int blocks, size_t lds, hipStream_t s);
bool ffnn_reg_eloc_launch_f16(int ke, const FfnnElocArgs &A, int G, int blocks, size_t lds, hipStream_t s);
size_t ffnn_reg_eloc_lds_bf16(int N, int ke, int m2p, int G);
size_t ffnn_reg_eloc_lds_f16(int N, int ke, int m2p, int G);
// Layer 2 can live in registers (8 waves x 32 output rows) for 16-bit operands
// with 128 <= m1p <= 512 and m2p <= 256.
static bool reg_path(int dtype, const FfnnDev &f)
{
    return (dtype == NQS_BF16 || dtype == NQS_F16) && f.m1p >= 128 && f.m1p <= 512 && f.m2p <= 256;
}

nqs_status deep_sample(nqs_model *m, const nqs_sample_cfg &cfg, int8_t *chain_state, int8_t *samples, float *logpsi,
                       uint64_t *n_accepted, const nqs_trace *trace, hipStream_t stream);
nqs_status deep_local_energy(nqs_model *m, const nqs_ham_desc &ham, const int8_t *samples, int64_t n, int dtype,
                             double *eloc, hipStream_t stream);

// Copy ready; *deep tells whether the network goes through the batched-GEMM path
// (any depth) instead of the two-layer kernels with an incremental first layer.
static nqs_status ffnn_mc_ready(nqs_model *m, int dtype, hipStream_t stream, bool *deep)
{
    if (dtype != NQS_F32 && dtype != NQS_BF16 && dtype != NQS_F16 && dtype != NQS_FP8_E4M3)
        return set_error(NQS_EUNSUPPORTED, "dense networks sample in F32, BF16, F16 or FP8_E4M3");
    nqs_status st = ensure_copy(m, dtype, stream);
    if (st != NQS_OK) return st;
    const FfnnDev &f = m->copies[dtype].ffnn;
    // the FP8 copy runs only the batched path (its layer products need whole E4M3 operand tiles)
    *deep = dtype == NQS_FP8_E4M3 || m->desc.n_layers != 2 || f.m1p > 512 ||
            (int64_t)f.widths[0] * f.m1p * (dtype == NQS_F32 ? 0 : 2) > 96 * 1024;
    return NQS_OK;
}

// The networks that the FP32 kernels take are those whose kRows rows fit; theirs are kRows32.
static size_t f32_spare(int dtype, const FfnnDev &f)
{
    if (dtype != NQS_F32) return 0;
    return sizeof(float) * ((size_t)kRows * (f.m1p + hs_pad<float>()) - (size_t)(f.m1p / 8) * kHBlock);
}

static size_t sample_lds_bytes(int dtype, int N, int m1p, int m2p)
{
    if (dtype == NQS_F32) return FfnnLds<float>::bytes(N, m1p, m2p);
    if (dtype == NQS_F16) return FfnnLds<_Float16>::bytes(N, m1p, m2p);
    return FfnnLds<__bf16>::bytes(N, m1p, m2p);
}

nqs_status ffnn_sample(nqs_model *m, const nqs_sample_cfg &cfg, int8_t *chain_state, int8_t *samples, float *logpsi,
                       uint64_t *n_accepted, const nqs_trace *trace, hipStream_t stream)
{
    bool deep = false;
    nqs_status st = ffnn_mc_ready(m, cfg.dtype, stream, &deep);
    if (st != NQS_OK) return st;
    if (deep || cfg.lanes_per_chain == -1) {
        if ((int64_t)(cfg.n_burnin + cfg.n_sweeps) * (cfg.sweep_size > 0 ? cfg.sweep_size : m->desc.n_visible) == 0) {
            if (cfg.init_chains) {
                st = launch_init_chains(chain_state, cfg.n_chains, m->desc.n_visible, cfg.move, cfg.seed,
                                        cfg.instance_id, cfg.chain_id_offset, stream);
                if (st != NQS_OK) return st;
            }
            if (n_accepted) return launch_zero_u64(n_accepted, cfg.n_chains, stream);
            return NQS_OK;
        }
        return deep_sample(m, cfg, chain_state, samples, logpsi, n_accepted, trace, stream);
    }
    const FfnnDev &f = m->copies[cfg.dtype].ffnn;
    const int N = f.widths[0];
    const int KE = f.n_layers >= 2 ? (f.widths[1] + 15) / 16 : 0;   // 16-wide fragments multiplied
    const size_t reg_lds = cfg.dtype == NQS_F16 ? ffnn_reg_sample_lds_f16(N, KE, f.m2p) : ffnn_reg_sample_lds_bf16(N, KE, f.m2p);
    const bool use_reg = reg_path(cfg.dtype, f) && reg_lds <= 160 * 1024;
    const size_t lds = use_reg ? reg_lds : sample_lds_bytes(cfg.dtype, N, f.m1p, f.m2p);
    if (lds + (use_reg ? 0 : f32_spare(cfg.dtype, f)) > 160 * 1024)
        return set_error(NQS_EUNSUPPORTED, "network too large for the LDS-resident sampler");
    if (cfg.init_chains) {
        st = launch_init_chains(chain_state, cfg.n_chains, N, cfg.move, cfg.seed, cfg.instance_id, cfg.chain_id_offset,
                                stream);
        if (st != NQS_OK) return st;
    }
    FfnnSampleArgs A;
    A.net = f;
    A.W2 = cfg.dtype == NQS_F32 ? (const void *)f.W2p : (const void *)f.W2c;
    A.W1t = cfg.dtype == NQS_F32 ? (const void *)f.W1tp : (const void *)f.W1ct;
    A.chain_state = chain_state;
    A.samples = samples;
    A.logpsi = logpsi;
    A.n_acc = (unsigned long long *)n_accepted;
    A.n_chains = cfg.n_chains;
    A.n_sweeps = cfg.n_sweeps;
    A.n_burnin = cfg.n_burnin;
    A.sweep_size = cfg.sweep_size > 0 ? cfg.sweep_size : N;
    A.refresh_sweeps = cfg.refresh_sweeps > 0 ? cfg.refresh_sweeps : 1;
    A.move = cfg.move;
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
    if ((int64_t)(cfg.n_burnin + cfg.n_sweeps) * A.sweep_size == 0) {
        if (n_accepted) return launch_zero_u64(n_accepted, cfg.n_chains, stream);
        return NQS_OK;
    }
    const int QK = (f.m1p + 63) / 64;
    if (use_reg) {
        // 8, 4, 2 or 1 chains per wave: the fewest whose blocks (one per CU, the LDS holds W1) all run at once.  A step
        // is a chain of latencies (draws, staging, products, decision) that shortens with the rows of a block:
        // 100-400-200, 100 exchange steps of 16,384, 4,096 and 1,024 chains take 568, 526 and 512 us with 8 per wave,
        // 325 us with 2 (4,096) and 264 us with 1 (1,024); 8 stays best where the blocks no longer fit (16,384 chains
        // with 4: 763 us).
        A.rpw = kRegRows / kRegWaves;
        while (A.rpw > 1 && (cfg.n_chains + kRegWaves * (A.rpw / 2) - 1) / (kRegWaves * (A.rpw / 2)) <= device_cus()) A.rpw /= 2;
        const int64_t blocks = (cfg.n_chains + kRegWaves * A.rpw - 1) / (kRegWaves * A.rpw);
        // With exchange moves about half the proposals swap equal spins: chains that
        // advance on their own decide those on the spot and fill every tile with
        // effective rows.  Flip moves are all effective, so the chains step together.
        const bool perchain = A.move == NQS_MOVE_EXCHANGE;
        const bool ok = cfg.dtype == NQS_F16 ? ffnn_reg_sample_launch_f16(KE, tr, perchain, A, (int)blocks, lds, stream)
                                             : ffnn_reg_sample_launch_bf16(KE, tr, perchain, A, (int)blocks, lds, stream);
        if (!ok) return set_error(NQS_EUNSUPPORTED, "first hidden width not supported by the register-resident sampler");
        NQS_HIP_TRY(hipGetLastError());
        return NQS_OK;
    }
    const int rows = cfg.dtype == NQS_F32 ? kRows32 : kRows;
    return ffnn_sample_dispatch(cfg.dtype, QK, tr, A, (int)((cfg.n_chains + rows - 1) / rows), lds, stream);
}

nqs_status ffnn_local_energy(nqs_model *m, const nqs_ham_desc &ham, const int8_t *samples, int64_t n, int dtype,
                             double *eloc, hipStream_t stream)
{
    bool deep = false;
    nqs_status st = ffnn_mc_ready(m, dtype, stream, &deep);
    if (st != NQS_OK) return st;
    if (m->desc.marshall && (m->desc.lat_dim != ham.dim || m->desc.lat_L != ham.L))
        return set_error(NQS_EINVAL, "Marshall lattice differs from the Hamiltonian lattice");
    if (deep) return deep_local_energy(m, ham, samples, n, dtype, eloc, stream);
    const FfnnDev &f = m->copies[dtype].ffnn;
    const int N = f.widths[0];
    size_t lds;
    // the register-resident kernel: W1 (16 KE columns) in LDS and groups of G samples (N < 8191 for the candidate
    // table), the G up to 8 whose rows the LDS holds that ends first: a group takes its passes and the time of about four
    // more, the CUs as many groups each.  100-400-200, BF16: groups of 2, 3, 4 and 5 samples take 22.5, 28.0, 33.7 and
    // 41.4 us; 1,025 samples end after 55.3 us with 5 (one group a CU; 58.7 with 4), 3,000 after 118 us with 4 (138 with 5).
    const int KE = f.n_layers >= 2 ? (f.widths[1] + 15) / 16 : 0;   // 16-wide fragments multiplied
    auto reg_lds_for = [&](int G) {
        return dtype == NQS_F16 ? ffnn_reg_eloc_lds_f16(N, KE, f.m2p, G) : ffnn_reg_eloc_lds_bf16(N, KE, f.m2p, G);
    };
    int reg_G = 1;
    double best = 0.0;
    const double rows = 1.0 + (ham.kind == NQS_TFIM ? N : 0.5 * ham.dim * N);   // of a sample, about
    for (int G = 1; G <= 8 && (G == 1 || reg_lds_for(G) <= 160 * 1024); ++G) {
        const int64_t rounds = ((n + G - 1) / G + device_cus() - 1) / device_cus();
        const double t = (double)rounds * (G * rows / kElocRows + 4.5);
        if (G == 1 || t < 0.97 * best) {
            reg_G = G;
            best = t;
        }
    }
    const size_t reg_lds = reg_path(dtype, f) ? reg_lds_for(reg_G) : 0;
    const bool use_reg = reg_path(dtype, f) && reg_lds <= 160 * 1024 && N < 8191;
    if (use_reg) lds = reg_lds;
    else if (dtype == NQS_F32) lds = ffnn_eloc_lds_bytes<float>(N, f.m1p, f.m2p);
    else if (dtype == NQS_F16) lds = ffnn_eloc_lds_bytes<_Float16>(N, f.m1p, f.m2p);
    else lds = ffnn_eloc_lds_bytes<__bf16>(N, f.m1p, f.m2p);
    if (lds + (use_reg ? 0 : f32_spare(dtype, f)) > 160 * 1024)
        return set_error(NQS_EUNSUPPORTED, "network too large for the local-energy kernel");
    if (m->desc.marshall && (m->desc.lat_dim != ham.dim || m->desc.lat_L != ham.L))
        return set_error(NQS_EINVAL, "Marshall lattice differs from the Hamiltonian lattice");
    FfnnElocArgs A;
    A.net = f;
    A.W2 = dtype == NQS_F32 ? (const void *)f.W2p : (const void *)f.W2c;
    A.W1t = dtype == NQS_F32 ? (const void *)f.W1tp : (const void *)f.W1ct;
    A.samples = samples;
    A.n = n;
    A.kind = ham.kind;
    A.dim = ham.dim;
    A.L = ham.L;
    A.pbc = ham.pbc;
    A.marshall = m->desc.marshall;
    A.J = ham.J;
    A.h = ham.h;
    A.eloc = eloc;
    const int QK = (f.m1p + 63) / 64;
    if (use_reg) {
        const int blocks = (int)std::min<int64_t>((n + reg_G - 1) / reg_G, device_cus());
        const bool ok = dtype == NQS_F16 ? ffnn_reg_eloc_launch_f16(KE, A, reg_G, blocks, lds, stream)
                                         : ffnn_reg_eloc_launch_bf16(KE, A, reg_G, blocks, lds, stream);
        if (!ok) return set_error(NQS_EUNSUPPORTED, "first hidden width not supported by the local-energy kernel");
        NQS_HIP_TRY(hipGetLastError());
        return NQS_OK;
    }
    const int blocks = (int)std::min<int64_t>(n, 256 * 4);
    return ffnn_eloc_dispatch(dtype, QK, A, blocks, lds, stream);
}

// ---- sample-space Gram matrix from the factors of O ----
//
// O of a dense layer is an outer product per sample: O_{W_l}[r][c] = delta_l[r] *
// a_{l-1}[c], O_{b_l}[r] = delta_l[r].  The factors (a few thousand floats per
// sample) are computed once; each column block of O is then expanded from them
// (a write-bound pass) instead of rerunning the forward and backward passes.

nqs_status ffnn_factors(nqs_model *m, const int8_t *samples, int64_t n, float *acts, float *dels, hipStream_t stream)
{
    nqs_status st = ensure_copy(m, NQS_F32, stream);
    if (st != NQS_OK) return st;
    const FfnnDev &net = m->copies[NQS_F32].ffnn;
    // networks that the gradient kernel does not take are refused here too
    size_t per = (size_t)((net.widths[0] + 3) & ~3), maxw = net.widths[0];
    for (int l = 1; l <= net.n_layers; ++l) {
        per += (size_t)((net.widths[l] + 3) & ~3);
        maxw = std::max(maxw, (size_t)net.widths[l]);
    }
    if (sizeof(float) * (per + 2 * ((maxw + 3) & ~(size_t)3)) > 160 * 1024)
        return set_error(NQS_EUNSUPPORTED, "network too wide for the gradient kernel");
    return factors_from(net, samples, n, acts, dels, nullptr, true, stream);
}

nqs_status ffnn_sample_gram(nqs_model *m, const int8_t *samples, int64_t n, int64_t chunk, float *T,
                            hipStream_t stream)
{
    nqs_status st = ensure_copy(m, NQS_F32, stream);
    if (st != NQS_OK) return st;
    const FfnnDev &net = m->copies[NQS_F32].ffnn;
    ExpandArgs E = expand_args(net);
    const int64_t sa = E.sa, sd = E.sd;
    const int64_t P = m->P;
    const size_t fa = (sizeof(float) * (size_t)n * sa + 255) & ~(size_t)255;
    const size_t fd = (sizeof(float) * (size_t)n * sd + 255) & ~(size_t)255;
    const size_t oc = (sizeof(float) * (size_t)n * chunk + 255) & ~(size_t)255;
    char *ws = (char *)workspace(fa + fd + oc + gram_workspace_bytes(n, chunk), stream);
    if (!ws) return set_error(NQS_ENOMEM, "workspace allocation failed");
    float *acts = (float *)ws, *dels = (float *)(ws + fa);
    E.acts = acts;
    E.dels = dels;
    float *Oc = (float *)(ws + fa + fd);

    st = ffnn_factors(m, samples, n, acts, dels, stream);
    if (st != NQS_OK) return st;

    if ((n + 15) / 16 > 65535) return set_error(NQS_EINVAL, "too many samples for the expansion grid");
    for (int64_t p0 = 0; p0 < P; p0 += chunk) {
        const int64_t p1 = std::min(P, p0 + chunk);
        st = expand_columns(E, n, p0, p1, Oc, stream);
        if (st != NQS_OK) return st;
        st = launch_gram_ws(Oc, n, p1 - p0, p0 == 0 ? 1 : 2, T, ws + fa + fd + oc, stream);
        if (st != NQS_OK) return st;
    }
    return NQS_OK;
}

}  // namespace nqs
