// Complex-parameter RBM: log psi = sum_i a_i s_i + sum_j log cosh(theta_j),
// theta = W s + b, a, b, W complex; the sampled distribution is |psi|^2 =
// exp(2 Re log psi).  Flipping site i multiplies psi by
//     exp(-2 a_i s_i) prod_j (C_ji - s_i t_j S_ji),
// C = cosh 2W, S = sinh 2W, t = tanh theta (all complex).
//
// Sampler: one chain per group of lanes, lanes over hidden units, complex
// (cosh theta, sinh theta) carried through accepted flips by the addition
// formulas and recomputed from W s + b every sweep (details at the kernel).
// Local energies: one sample per workgroup, one thread per site, the complex
// flip ratios summed in FP64 (real and imaginary parts).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "common.h"
#include "crbm_math.h"
#include "internal.h"

namespace nqs {

constexpr int kCrbmThreads = 256;

// ---- copy ----

__global__ void crbm_build_kernel(const double *__restrict__ master, int N, int M, int dtype, CrbmDev d)
{
    const int64_t P = N + M + (int64_t)M * N;
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q < N) {
        d.a[q] = make_float2((float)round_to_dtype(master[q], dtype), (float)round_to_dtype(master[P + q], dtype));
        d.a2[q] = (float)(4.0 * round_to_dtype(master[q], dtype) / 0.69314718055994531);
    } else if (q < N + M) {
        d.b[q - N] = make_float2((float)round_to_dtype(master[q], dtype), (float)round_to_dtype(master[P + q], dtype));
    } else if (q < P) {
        const int64_t r = q - N - M;
        const int j = (int)(r / N), i = (int)(r - (int64_t)j * N);
        const double wr = round_to_dtype(master[q], dtype), wi = round_to_dtype(master[P + q], dtype);
        d.Wt[(int64_t)i * M + j] = make_float2((float)wr, (float)wi);
        // cosh 2w = cosh 2x cos 2y + i sinh 2x sin 2y; sinh 2w = sinh 2x cos 2y + i cosh 2x sin 2y
        const double ch = cosh(2.0 * wr), sh = sinh(2.0 * wr), c = cos(2.0 * wi), s = sin(2.0 * wi);
        const float4 cs = make_float4((float)(ch * c), (float)(sh * s), (float)(sh * c), (float)(ch * s));
        d.CS[(int64_t)i * M + j] = cs;
        d.CSt[(int64_t)j * N + i] = cs;
    } else if (q == P) {
        d.CS[(int64_t)N * M] = make_float4(1.0f, 0.0f, 0.0f, 0.0f);   // neutral entry for lanes past the last unit
    }
}

nqs_status crbm_build_copy(nqs_model *m, int dtype, hipStream_t stream)
{
    if (dtype == NQS_FP8_E4M3) return set_error(NQS_EUNSUPPORTED, "no FP8 copy of the complex RBM");
    const int N = m->desc.n_visible, M = m->desc.widths[0];
    Copy &c = m->copies[dtype];
    CrbmDev &d = c.crbm;
    d.N = N;
    d.M = M;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t nm = (size_t)N * M;
    const size_t bytes = al(sizeof(float2) * N) + al(sizeof(float) * N) + al(sizeof(float2) * M) +
                         al(sizeof(float2) * nm) + al(sizeof(float4) * (nm + 1)) + al(sizeof(float4) * nm);
    if (!c.block) NQS_HIP_TRY(hipMalloc(&c.block, bytes));
    char *p = (char *)c.block;
    d.a = (float2 *)p;
    p += al(sizeof(float2) * N);
    d.a2 = (float *)p;
    p += al(sizeof(float) * N);
    d.b = (float2 *)p;
    p += al(sizeof(float2) * M);
    d.Wt = (float2 *)p;
    p += al(sizeof(float2) * nm);
    d.CS = (float4 *)p;
    p += al(sizeof(float4) * (nm + 1));
    d.CSt = (float4 *)p;
    const int64_t P = N + M + (int64_t)nm;
    hipLaunchKernelGGL(crbm_build_kernel, dim3((unsigned)((P + 1 + 255) / 256)), dim3(256), 0, stream, m->master, N,
                       M, dtype, d);
    NQS_HIP_TRY(hipGetLastError());
    c.valid = true;
    return NQS_OK;
}

// ---- sampler ----
//
// One chain per group of G lanes (G = 16, 32 or 64); lane g of the group owns
// hidden units j = g + qG, q < K, and spin word g (32 spins per word).  Per
// unit the chain keeps complex (c_j, s_j) proportional to (cosh theta_j,
// sinh theta_j), with c = 1 after each refresh, and per lane the running
// log2 of prod_q |c_q|^2.  With C = cosh 2W_ji and S = sinh 2W_ji, flipping
// site i gives
//   n_j = c_j C - s_i s_j S = c_j cosh(theta_j - 2 s_i W_ji) / cosh theta_j,
//   log2 |psi(s')/psi(s)|^2 = -4 Re(a_i) s_i / ln 2 + sum_j [log2 |n_j|^2 - log2 |c_j|^2],
// and an accepted flip sets c_j <- n_j, s_j <- s_j C - s_i c_j S.  The move is
// accepted iff log2 u < that log-ratio.  The squared moduli of a lane are
// multiplied (renormalised every four factors) and take one logarithm.  The
// (C, S) column of the next proposal is loaded while the current one is
// decided; the table sits in LDS when it fits, else it is read through L2.
//
// With one or two waves per SIMD a step is its wave's chain of instructions (8.3
// cycles where one needs the one before): broadcasts run two proposals ahead, the
// next proposal's spin is read before this one's decision and corrected for it,
// all but the last FMA of the move's sinh is formed while the decision's sum is
// under way, and the steps between two refreshes or draws run without tests.
// 3,000 chains of 16, 64 and 100 sites with as many units: 517, 839 and 755 ns a
// step before (the second with 128 units), 378, 757 and 673 ns now.

struct CrbmSampleArgs {
    CrbmDev net;
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

constexpr int kCrbmMaxK = 8;

// theta = W s + b from the spin words; c = 1, s = tanh theta.  Returns
// Re log psi (FP32) when want_f (uniform across the group), else 0.
template <int G, int K>
__device__ __forceinline__ float crbm_refresh(const CrbmDev &net, uint32_t word, int gl, float2 (&c)[K],
                                              float2 (&sh)[K], bool want_f)
{
    const int N = net.N, M = net.M;
    constexpr int CH = K >= 6 ? 2 : 4;   // sites whose W rows are in flight together
    float2 th[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int j = gl + k * G;
        th[k] = j < M ? net.b[j] : make_float2(0.0f, 0.0f);
    }
    const int jl = gl + (K - 1) * G;
    const int jlast = jl < M ? jl : M - 1;          // clamp the tail slot to a valid column
    const float wlast = jl < M ? 1.0f : 0.0f;
    float as = 0.0f;
    const int NW = (N + 31) >> 5;
    for (int w = 0; w < NW; ++w) {
        const uint32_t bits = group_bcast<G>(word, w);
        const int i0 = w << 5;
        const int nb = min(32, N - i0);
        int bb = 0;
        for (; bb + CH <= nb; bb += CH) {
            float2 wv[CH][K];
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                const float2 *wrow = net.Wt + (size_t)(i0 + bb + q) * M;
#pragma unroll
                for (int k = 0; k < K - 1; ++k) wv[q][k] = wrow[gl + k * G];
                wv[q][K - 1] = wrow[jlast];
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                const float s = ((bits >> (bb + q)) & 1u) ? 1.0f : -1.0f;
                as = fmaf(net.a[i0 + bb + q].x, s, as);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const float sw = k == K - 1 ? s * wlast : s;
                    th[k].x = fmaf(wv[q][k].x, sw, th[k].x);
                    th[k].y = fmaf(wv[q][k].y, sw, th[k].y);
                }
            }
        }
        for (; bb < nb; ++bb) {
            const float2 *wrow = net.Wt + (size_t)(i0 + bb) * M;
            const float s = ((bits >> bb) & 1u) ? 1.0f : -1.0f;
            as = fmaf(net.a[i0 + bb].x, s, as);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float2 wk = wrow[k == K - 1 ? jlast : gl + k * G];
                const float sw = k == K - 1 ? s * wlast : s;
                th[k].x = fmaf(wk.x, sw, th[k].x);
                th[k].y = fmaf(wk.y, sw, th[k].y);
            }
        }
    }
    float lc = 0.0f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        c[k] = make_float2(1.0f, 0.0f);
        sh[k] = ctanh(th[k]);
        if (want_f && (k < K - 1 || jl < M)) lc += clogcosh_re(th[k]);
    }
    return want_f ? as + group_sum_uniform<G>(lc) : 0.0f;
}

// Proposal (batch start + g) for lane g of a group: site, u bits, log2 u and
// the negative visible-bias term, -4 Re(a_i) / ln 2.
struct CrbmProp {
    uint32_t i, ub;
    float l2u, a2;
};

__device__ __forceinline__ CrbmProp crbm_prop(const CrbmDev &net, uint64_t step, uint32_t gid, uint32_t inst,
                                              uint32_t key0, uint32_t key1)
{
    const Block4 rb = philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), gid, inst << 8, key0, key1);
    CrbmProp pb;
    pb.i = (uint32_t)index_from_word(rb.r0, net.N);
    pb.ub = rb.r2 >> 8;
    pb.l2u = __builtin_amdgcn_logf((float)pb.ub * 5.9604644775390625e-8f);   // log2 u, u = ub 2^-24
    pb.a2 = -net.a2[pb.i];
    return pb;
}

template <int G, int K, bool LDS_TAB>
__global__ void __launch_bounds__(G == 16 ? 256 : 512) crbm_sample_kernel(CrbmSampleArgs A)
{
    extern __shared__ float4 s_ctab[];
    const int N = A.net.N, M = A.net.M;
    if constexpr (LDS_TAB) {
        const int tot = N * M + 1;   // includes the neutral entry
        for (int k = threadIdx.x; k < tot; k += blockDim.x) s_ctab[k] = A.net.CS[k];
        __syncthreads();
    }
    const int cpb = blockDim.x / G;
    const int gl = threadIdx.x % G;
    const int64_t c = (int64_t)blockIdx.x * cpb + threadIdx.x / G;
    if (c >= A.n_chains) return;   // whole groups leave together; no barrier follows

    const uint32_t gid = A.chain_id_offset + (uint32_t)c;
    const uint32_t key0 = (uint32_t)A.seed, key1 = (uint32_t)(A.seed >> 32);
    const int NW = (N + 31) >> 5;
    const bool last_ok = gl + (K - 1) * G < M;
    const int base4 = ((int)(threadIdx.x & 63) & ~(G - 1)) << 2;
    // byte offsets of a column's entries of this lane: its first, and its last or the neutral entry behind the table
    const int col_step = 16 * M, col_first = 16 * gl;
    const int last_step = last_ok ? 16 * M : 0, last_first = last_ok ? 16 * (gl + (K - 1) * G) : 16 * N * M;

    uint32_t word = 0;
    if (gl < NW) {
        const int nb = min(32, N - gl * 32);
        const int8_t *src = A.chain_state + (size_t)c * N + gl * 32;
        for (int bb = 0; bb < nb; ++bb) word |= (src[bb] > 0 ? 1u : 0u) << bb;
    }
    float2 cc[K], sh[K];
    crbm_refresh<G, K>(A.net, word, gl, cc, sh, false);
    float lpart = 0.0f;

    const int sw = A.sweep_size;
    const int64_t total = (int64_t)(A.n_burnin + A.n_sweeps) * sw;
    const bool traced = c < A.n_traced;
    unsigned long long acc = 0;
    int in_sweep = 0;
    int64_t sweep = 0;

    // proposal pipeline: `cur` covers steps [base, base+G), `nxt` the next G; a step starts with its own and the next
    // proposal in registers and broadcasts the one after
    uint64_t base = A.step_offset;
    CrbmProp cur = crbm_prop(A.net, base + gl, gid, A.inst, key0, key1);
    CrbmProp nxt = crbm_prop(A.net, base + G + gl, gid, A.inst, key0, key1);
    int p = 0;
    int i_c = (int)group_bcast<G>(cur.i, 0), i_n = (int)group_bcast<G>(cur.i, 1);
    float l2u_c = __uint_as_float(group_bcast<G>(__float_as_uint(cur.l2u), 0));
    float l2u_n = __uint_as_float(group_bcast<G>(__float_as_uint(cur.l2u), 1));
    float a2_c = __uint_as_float(group_bcast<G>(__float_as_uint(cur.a2), 0));
    float a2_n = __uint_as_float(group_bcast<G>(__float_as_uint(cur.a2), 1));
    uint32_t smask = (group_bcast<G>(~word, i_c >> 5) >> (i_c & 31)) << 31;   // sign of site i_c's spin: 0 up, 2^31 down
    float4 csA[K], csB[K];
    auto column = [&](int i, float4 (&cs)[K]) {
        const unsigned char *t = reinterpret_cast<const unsigned char *>(LDS_TAB ? s_ctab : A.net.CS);
        const float4 *col = reinterpret_cast<const float4 *>(t + (i * col_step + col_first));
#pragma unroll
        for (int q = 0; q < K - 1; ++q) cs[q] = col[q * G];
        cs[K - 1] = *reinterpret_cast<const float4 *>(t + (i * last_step + last_first));
    };
    column(i_c, csA);

    // one proposal: evaluate with cs_c (column of i_c), prefetch the next column into cs_n
    auto step = [&](int64_t k, float4 (&cs_c)[K], float4 (&cs_n)[K]) {
        column(i_n, cs_n);
        // the spin of the next proposal's site before this one's decision, and the proposal after the next
        const uint32_t smask_b = (~group_bcast4<G>(word, base4, (i_n >> 3) & ~3) >> (i_n & 31)) << 31;
        // the last lanes' proposals after the next are the next batch's first
        const bool in_cur = p + 2 < G;
        const int pl = (in_cur ? p + 2 : p + 2 - G) << 2;
        const int i_f = (int)group_bcast4<G>(in_cur ? cur.i : nxt.i, base4, pl);
        const float l2u_f = __uint_as_float(group_bcast4<G>(__float_as_uint(in_cur ? cur.l2u : nxt.l2u), base4, pl));
        const float a2_f = __uint_as_float(group_bcast4<G>(__float_as_uint(in_cur ? cur.a2 : nxt.a2), base4, pl));

        // proposal k: flip site i_c
        const float si = __uint_as_float(0x3F800000u | smask);
        uint32_t flip = gl == (i_c >> 5) ? 1u << (i_c & 31) : 0u, same = i_n == i_c ? 0x80000000u : 0u;
        asm volatile("" : "+v"(flip), "+v"(same));                         // formed before the decision
        float2 nn[K], ns[K];
        float prod = 1.0f;
        int e2 = 0;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const float4 t = cs_c[q];
            const float spx = si * t.z, spy = si * t.w;                    // s_i S
            float nx = fmaf(cc[q].x, t.x, -cc[q].y * t.y);                 // c C
            float ny = fmaf(cc[q].x, t.y, cc[q].y * t.x);
            nx = fmaf(-sh[q].x, spx, fmaf(sh[q].y, spy, nx));               // - s (s_i S)
            ny = fmaf(-sh[q].x, spy, fmaf(-sh[q].y, spx, ny));
            nn[q] = make_float2(nx, ny);
            prod *= fmaf(nx, nx, ny * ny);
            if ((q & 3) == 3 && q + 1 < K) {
                int e;
                prod = frexpf(prod, &e);
                e2 += e;
            }
        }
        const float lnew = __builtin_amdgcn_logf(prod) + (float)e2;     // log2 prod |n|^2
        float d2 = lnew - lpart;
        // the move's s_j C - s_i c_j S, all but its last FMA, while the sum over the lanes is under way
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const float4 t = cs_c[q];
            const float spx = si * t.z, spy = si * t.w;
            float sx = fmaf(sh[q].x, t.x, -sh[q].y * t.y);                  // s C
            float sy = fmaf(sh[q].x, t.y, sh[q].y * t.x);
            ns[q] = make_float2(fmaf(cc[q].y, spy, sx), fmaf(-cc[q].y, spx, sy));   // - c (s_i S), first half
            asm volatile("" : "+v"(ns[q].x), "+v"(ns[q].y));               // not sunk below the decision
        }
        d2 = group_sum_uniform<G>(d2) + __uint_as_float(__float_as_uint(a2_c) ^ smask);
        const bool accept = l2u_c < d2;                                 // NaN rejects
        if (accept) {
#pragma unroll
            for (int q = 0; q < K; ++q) {
                const float4 t = cs_c[q];
                const float spx = si * t.z, spy = si * t.w;
                sh[q] = make_float2(fmaf(-cc[q].x, spx, ns[q].x), fmaf(-cc[q].x, spy, ns[q].y));
                cc[q] = nn[q];
            }
            lpart = lnew;
            word ^= flip;
            ++acc;
        }
        if (traced) {
            const uint32_t ub_c = group_bcast<G>(cur.ub, p);
            if (gl == 0) {
                const size_t idx = (size_t)c * (size_t)total + (size_t)k;
                A.tr_site[idx] = i_c | (0xFFFF << 16);
                A.tr_ubits[idx] = ub_c;
                A.tr_delta[idx] = d2 * 0.69314718055994531f;
                A.tr_acc[idx] = accept ? 1 : 0;
            }
        }
        // advance the pipeline
        smask = smask_b ^ (accept ? same : 0u);
        i_c = i_n;
        l2u_c = l2u_n;
        a2_c = a2_n;
        i_n = i_f;
        l2u_n = l2u_f;
        a2_n = a2_f;
        ++p;
    };

    for (int64_t k = 0; k < total;) {
        // the steps up to the end of the sweep or of the drawn proposals
        const int run = min(sw - in_sweep, G - p);
        int r = 0;
        for (; r + 1 < run; r += 2) {
            step(k + r, csA, csB);
            step(k + r + 1, csB, csA);
        }
        if (r < run) {
            step(k + r, csA, csB);
#pragma unroll
            for (int q = 0; q < K; ++q) csA[q] = csB[q];
        }
        k += run;
        in_sweep += run;
        if (p == G) {
            p = 0;
            base += G;
            cur = nxt;
            nxt = crbm_prop(A.net, base + G + gl, gid, A.inst, key0, key1);
        }
        if (in_sweep == sw) {
            in_sweep = 0;
            const int64_t out = sweep - A.n_burnin;
            const bool need_f = A.logpsi != nullptr && out >= 0;
            const float f = crbm_refresh<G, K>(A.net, word, gl, cc, sh, need_f);
            lpart = 0.0f;
            if (out >= 0) {
                if (A.samples && gl < NW) {
                    int8_t *dst = A.samples + ((size_t)out * A.n_chains + c) * N + gl * 32;
                    const int nb = min(32, N - gl * 32);
                    for (int bb = 0; bb < nb; ++bb) dst[bb] = ((word >> bb) & 1u) ? 1 : -1;
                }
                if (A.logpsi && gl == 0) A.logpsi[(size_t)out * A.n_chains + c] = f;
            }
            ++sweep;
        }
    }

    if (gl < NW) {
        int8_t *dst = A.chain_state + (size_t)c * N + gl * 32;
        const int nb = min(32, N - gl * 32);
        for (int bb = 0; bb < nb; ++bb) dst[bb] = ((word >> bb) & 1u) ? 1 : -1;
    }
    if (A.n_acc && gl == 0) A.n_acc[c] = acc;
}

// ---- TFIM local energies, complex: B samples per workgroup ----
//
// Per sample: t = tanh theta in LDS; one thread per site and kCrbmSB samples
// forms their complex flip ratios, exp(-2 a_i s_i) prod_j (C - s_i t_j S), with
// frexp renormalisation every 8 factors, and stores them in FP64; then one wave
// per sample sums ratios and diagonal bonds in a fixed order.  A table element
// (W for theta, (C, S) for the ratios) is read once per kCrbmSB samples, mostly
// from L1 where the workgroup's other samples want it too.
//
// Bound by the vector unit (about 12 instructions per sample, site and unit)
// once enough waves hide a factor's chain of dependent products.  100 x 200,
// 30,000 samples: 277 us with four samples per thread and eight per workgroup
// (12 waves on a CU); 734 us with sixteen samples per thread (4 waves, the table
// elements one at a time).
constexpr int kCrbmSB = 4;   // samples per thread (1 where the LDS holds fewer)

__device__ inline double crbm_bonds(const float *s, int i, int dim, int L, int pbc)
{
    const float si = s[i];
    double dg = 0.0;   // bonds to the right / below, each counted once
    if (dim == 1) {
        if (i + 1 < L) dg += (double)(si * s[i + 1]);
        else if (pbc) dg += (double)(si * s[0]);
    } else {
        const int x = i / L, y = i - (i / L) * L;
        if (x + 1 < L) dg += (double)(si * s[(x + 1) * L + y]);
        else if (pbc) dg += (double)(si * s[y]);
        if (y + 1 < L) dg += (double)(si * s[x * L + y + 1]);
        else if (pbc) dg += (double)(si * s[x * L]);
    }
    return dg;
}

__host__ __device__ inline size_t crbm_eloc_lds(int B, int N, int M)
{
    return sizeof(double2) * (size_t)B * N + sizeof(float2) * (size_t)B * M + sizeof(float) * (size_t)B * N;
}

template <int SB>
__global__ void __launch_bounds__(256) crbm_eloc_tfim_kernel(CrbmDev net, const int8_t *__restrict__ samples,
                                                             int64_t n, int B, int dim, int L, int pbc, double J,
                                                             double h, double *__restrict__ eloc_re,
                                                             double *__restrict__ eloc_im)
{
    extern __shared__ double2 crbm_esm[];
    const int N = net.N, M = net.M, tid = threadIdx.x, nt = blockDim.x;
    double2 *rat = crbm_esm;                                             // [B][N]
    float2 *tt = reinterpret_cast<float2 *>(rat + (size_t)B * N);       // [B][M]
    float *s = reinterpret_cast<float *>(tt + (size_t)B * M);           // [B][N]
    for (int64_t k0 = (int64_t)blockIdx.x * B; k0 < n; k0 += (int64_t)gridDim.x * B) {
        const int nb = (int)(n - k0 < B ? n - k0 : B);
        const int ng = (nb + SB - 1) / SB;   // groups of SB samples
        for (int e = tid; e < B * N; e += nt) {
            const int bb = e / N, i = e - bb * N;
            s[e] = bb < nb ? (float)samples[(k0 + bb) * N + i] : 1.0f;
        }
        __syncthreads();
        for (int t = tid; t < M * ng; t += nt) {
            const int g = t / M, j = t - g * M;
            const float *sg = s + g * SB * N;
            float2 th[SB];
            const float2 bj = net.b[j];
#pragma unroll
            for (int bb = 0; bb < SB; ++bb) th[bb] = bj;
#pragma unroll 8
            for (int i = 0; i < N; ++i) {
                const float2 w = net.Wt[(int64_t)i * M + j];
#pragma unroll
                for (int bb = 0; bb < SB; ++bb) {
                    const float sb = sg[bb * N + i];
                    th[bb].x = fmaf(w.x, sb, th[bb].x);
                    th[bb].y = fmaf(w.y, sb, th[bb].y);
                }
            }
#pragma unroll
            for (int bb = 0; bb < SB; ++bb) tt[(g * SB + bb) * M + j] = ctanh(th[bb]);
        }
        __syncthreads();
        for (int t = tid; t < N * ng; t += nt) {
            const int g = t / N, i = t - g * N;
            const float2 *tg = tt + g * SB * M;
            float2 pr[SB];
            int e2[SB];
            float si[SB];
#pragma unroll
            for (int bb = 0; bb < SB; ++bb) {
                pr[bb] = make_float2(1.0f, 0.0f);
                e2[bb] = 0;
                si[bb] = s[(g * SB + bb) * N + i];
            }
            auto factor = [&](float4 cs, int j) {
#pragma unroll
                for (int bb = 0; bb < SB; ++bb) {
                    const float2 ts = cmul(tg[bb * M + j], make_float2(cs.z, cs.w));
                    pr[bb] = cmul(pr[bb], make_float2(fmaf(-si[bb], ts.x, cs.x), fmaf(-si[bb], ts.y, cs.y)));
                }
            };
            int j = 0;
            for (; j + 8 <= M; j += 8) {
                float4 cs[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) cs[u] = net.CSt[(int64_t)(j + u) * N + i];
#pragma unroll
                for (int u = 0; u < 8; ++u) factor(cs[u], j + u);
#pragma unroll
                for (int bb = 0; bb < SB; ++bb) {
                    int e;
                    (void)frexpf(fmaxf(fabsf(pr[bb].x), fabsf(pr[bb].y)), &e);
                    pr[bb].x = ldexpf(pr[bb].x, -e);
                    pr[bb].y = ldexpf(pr[bb].y, -e);
                    e2[bb] += e;
                }
            }
            for (; j < M; ++j) factor(net.CSt[(int64_t)j * N + i], j);
            // exp(-2 a_i s) for both spins
            const float2 ai = net.a[i];
            double mag[2], sn[2], cn[2];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const float sv = v ? 1.0f : -1.0f;
                mag[v] = exp(-2.0 * (double)ai.x * sv);
                sincos(-2.0 * (double)ai.y * sv, &sn[v], &cn[v]);
            }
#pragma unroll
            for (int bb = 0; bb < SB; ++bb) {
                const bool up = si[bb] > 0.0f;
                const double mg = (up ? mag[1] : mag[0]) * ldexp(1.0, e2[bb]);
                const double pre = mg * (up ? cn[1] : cn[0]), pim = mg * (up ? sn[1] : sn[0]);
                rat[(g * SB + bb) * N + i] = make_double2(pre * pr[bb].x - pim * pr[bb].y, pre * pr[bb].y + pim * pr[bb].x);
            }
        }
        __syncthreads();
        const int wave = tid >> 6, lane = tid & 63, nw = nt >> 6;
        for (int bb = wave; bb < nb; bb += nw) {
            double re = 0.0, im = 0.0, dg = 0.0;
            for (int i = lane; i < N; i += 64) {
                re += rat[bb * N + i].x;
                im += rat[bb * N + i].y;
                dg += crbm_bonds(s + bb * N, i, dim, L, pbc);
            }
            re = group_sum<64>(re);
            im = group_sum<64>(im);
            dg = group_sum<64>(dg);
            if (lane == 0) {
                eloc_re[k0 + bb] = J * dg + h * re;
                if (eloc_im) eloc_im[k0 + bb] = h * im;
            }
        }
        __syncthreads();
    }
}

// ---- host ----

template <int G, int K>
static void crbm_launch_gk(const CrbmSampleArgs &A, int64_t blocks, int threads, size_t lds_bytes, hipStream_t s)
{
    if (lds_bytes) {
        allow_lds(crbm_sample_kernel<G, K, true>, lds_bytes);
        hipLaunchKernelGGL((crbm_sample_kernel<G, K, true>), dim3((unsigned)blocks), dim3(threads), lds_bytes, s, A);
    } else {
        hipLaunchKernelGGL((crbm_sample_kernel<G, K, false>), dim3((unsigned)blocks), dim3(threads), 0, s, A);
    }
}

template <int G>
static void crbm_launch_g(int K, const CrbmSampleArgs &A, int64_t blocks, int threads, size_t lds_bytes, hipStream_t s)
{
    switch (K) {
    case 1: crbm_launch_gk<G, 1>(A, blocks, threads, lds_bytes, s); break;
    case 2: crbm_launch_gk<G, 2>(A, blocks, threads, lds_bytes, s); break;
    case 3: crbm_launch_gk<G, 3>(A, blocks, threads, lds_bytes, s); break;
    case 4: crbm_launch_gk<G, 4>(A, blocks, threads, lds_bytes, s); break;
    case 5: crbm_launch_gk<G, 5>(A, blocks, threads, lds_bytes, s); break;
    case 6: crbm_launch_gk<G, 6>(A, blocks, threads, lds_bytes, s); break;
    case 7: crbm_launch_gk<G, 7>(A, blocks, threads, lds_bytes, s); break;
    default: crbm_launch_gk<G, 8>(A, blocks, threads, lds_bytes, s); break;
    }
}

nqs_status crbm_sample(nqs_model *m, const nqs_sample_cfg &cfg, int8_t *chain_state, int8_t *samples, float *logpsi,
                       uint64_t *n_accepted, const nqs_trace *trace, hipStream_t stream)
{
    nqs_status st = ensure_copy(m, cfg.dtype, stream);
    if (st != NQS_OK) return st;
    const CrbmDev &net = m->copies[cfg.dtype].crbm;
    const int N = net.N, M = net.M;
    // launch shape: lanes per chain G, hidden units per lane K = ceil(M / G) <= 8
    int G = cfg.lanes_per_chain;
    if (G == 0) {
        G = 16;
        while (G < 64 && ((N + 31) / 32 > G || (M + G - 1) / G > kCrbmMaxK)) G *= 2;
    } else if (G != 16 && G != 32 && G != 64) {
        return set_error(NQS_EUNSUPPORTED, "complex RBM sampler: lanes_per_chain must be 0, 16, 32 or 64");
    }
    if ((N + 31) / 32 > G) return set_error(NQS_EUNSUPPORTED, "complex RBM sampler: too many sites (N <= 32 G)");
    const int K = (M + G - 1) / G;
    if (K > kCrbmMaxK) return set_error(NQS_EUNSUPPORTED, "complex RBM sampler: at most 8 hidden units per lane (M <= 512)");
    if (cfg.init_chains) {
        st = launch_init_chains(chain_state, cfg.n_chains, N, NQS_MOVE_FLIP, cfg.seed, cfg.instance_id,
                                cfg.chain_id_offset, stream);
        if (st != NQS_OK) return st;
    }
    if (cfg.n_chains == 0) return NQS_OK;
    CrbmSampleArgs A;
    A.net = net;
    A.chain_state = chain_state;
    A.samples = samples;
    A.logpsi = logpsi;
    A.n_acc = (unsigned long long *)n_accepted;
    A.n_chains = cfg.n_chains;
    A.n_sweeps = cfg.n_sweeps;
    A.n_burnin = cfg.n_burnin;
    A.sweep_size = cfg.sweep_size > 0 ? cfg.sweep_size : N;
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
    // one LDS copy of the table per block when it fits; spread the chains over every CU
    constexpr size_t kLds = 160 * 1024;
    const size_t tab_bytes = sizeof(float4) * ((size_t)N * M + 1);
    const bool lds = tab_bytes <= kLds;
    const int max_threads = G == 16 ? 256 : 512;
    const int blocks_per_cu = lds ? (int)std::max<size_t>(1, std::min<size_t>(8, kLds / tab_bytes)) : 8;
    const int64_t slots = (int64_t)device_cus() * blocks_per_cu;
    // whole waves once there are more chains than SIMDs: 100 x 200, G = 32, ten sweeps and two of burn-in, 2,048 chains
    // 1,231 us with one chain per wave, 905 with two (1,024 chains: 893 us with one)
    const int64_t least = cfg.n_chains > 4 * (int64_t)device_cus() ? 64 / G : 1;
    const int cpb = (int)std::min<int64_t>(max_threads / G, std::max<int64_t>(least, (cfg.n_chains + slots - 1) / slots));
    const int64_t blocks = (cfg.n_chains + cpb - 1) / cpb;
    if (blocks > INT32_MAX) return set_error(NQS_EINVAL, "too many chains");
    const size_t lds_bytes = lds ? tab_bytes : 0;
    switch (G) {
    case 16: crbm_launch_g<16>(K, A, blocks, cpb * G, lds_bytes, stream); break;
    case 32: crbm_launch_g<32>(K, A, blocks, cpb * G, lds_bytes, stream); break;
    default: crbm_launch_g<64>(K, A, blocks, cpb * G, lds_bytes, stream); break;
    }
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

nqs_status crbm_local_energy(nqs_model *m, const nqs_ham_desc &ham, const int8_t *samples, int64_t n, int dtype,
                             double *eloc_re, double *eloc_im, hipStream_t stream)
{
    if (ham.kind != NQS_TFIM) return set_error(NQS_EUNSUPPORTED, "complex RBM local energies: TFIM");
    nqs_status st = ensure_copy(m, dtype, stream);
    if (st != NQS_OK) return st;
    const CrbmDev &net = m->copies[dtype].crbm;
    // samples per workgroup: two groups, one, or one sample, whose LDS stays within 64 KB, else 160 KB; threads for two
    // groups' sites (30,000 samples of 64 sites, 128 units: 120 us with 128 threads, 156 with 256; 100 sites, 200 units:
    // 323 and 277 us)
    int B = 2 * kCrbmSB;
    if (crbm_eloc_lds(B, net.N, net.M) > 64 * 1024) B = kCrbmSB;
    if (crbm_eloc_lds(B, net.N, net.M) > 160 * 1024) B = 1;
    const size_t lds = crbm_eloc_lds(B, net.N, net.M);
    if (lds > 160 * 1024) return set_error(NQS_EUNSUPPORTED, "complex RBM too large for the local-energy kernel");
    if (n == 0) return NQS_OK;
    const int threads = 2 * net.N <= 128 ? 128 : 256;
    const int64_t blocks = std::min<int64_t>((n + B - 1) / B, (int64_t)device_cus() * 32);
    auto launch = [&](auto kernel) {
        allow_lds(kernel, lds);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), lds, stream, net, samples, n, B, ham.dim, ham.L,
                           ham.pbc, ham.J, ham.h, eloc_re, eloc_im);
    };
    if (B == 1) launch(crbm_eloc_tfim_kernel<1>);
    else launch(crbm_eloc_tfim_kernel<kCrbmSB>);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

}  // namespace nqs
