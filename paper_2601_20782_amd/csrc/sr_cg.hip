// Jacobi-preconditioned conjugate gradients for (T + shift) y = eps - mean(eps) in one cooperative launch, T held in
// registers (n up to 4096; above it, up to 5120, the columns that do not fit are read again each iteration).
//
// As two launches per iteration the solve spent 31 us of an n = 4096 iteration on reading T (67 MB) at 256
// wavefronts' worth of loads in flight, on one block's vector updates, and on the gaps between launches.  But 67 MB
// are half of the chip's 128 MB of vector registers: a block of 1024 threads per CU keeps its 16 rows of T (64 of the
// 128 registers that a thread may have; the form for n up to 4096 spills 12 others, the one above it 11) from the first
// iteration to the last.  What an iteration then has to move is T p: every block
// publishes its 16 values, reads all n of them, and repeats the scalar sums and the updates of r, z and p for all n
// elements in the same order, so that every block holds the same bits and takes the same decisions.  One exchange an
// iteration, no other communication.
//
// Exchange: a value is published with one 8-byte device-scope store into a slot that held a NaN of a payload which
// no arithmetic produces, and a reader polls the slot until it holds something else; the data is its own flag, and no
// fence is needed.  Three buffers in turn: when a block has read all values of iteration k, every block has read all
// of k - 1 (each publishes k after that), so it resets its own slots of that buffer, before it publishes k + 1; a
// block polls them again in iteration k + 2, after it has seen all of k + 1.
//
// The launch is cooperative (all blocks resident) and every wait is bounded: a block that waits too long gives up,
// the others follow, and the caller solves with separate launches.
//
// Bound by the exchange: an iteration takes 4.4 us at n = 64, 4.7 at n = 1024 (16.4 as two launches), 7.4 at n = 4096
// (36) and 17.9 at n = 5000 (47), of which the sums by DPP instead of shuffles through LDS saved 1.3 to 1.7.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "common.h"
#include "internal.h"
#include "nqs.h"
#include "nqs_probe.h"

namespace nqs {

constexpr int kCgThreads = 1024;
constexpr int kCgWaves = kCgThreads / 64;
constexpr int kCgGroups = 4;                 // column groups; the other kCgWaves / kCgGroups = 4 are row groups
constexpr unsigned long long kCgEmpty = 0x7FF8A5C3D2E1F00Full;
// Beyond 5120 unknowns more than two fifths of T would be read again each iteration, and two launches are as good
// (n = 8192: 82 us an iteration this way, 87 us as two launches).
constexpr int64_t kCgMax = 5120;
constexpr int kCgPolls = 1 << 21;            // before a block gives up (seconds)

// of the calling thread: polls of its later solves (0: kCgPolls), and whether its last one was one launch (-1: none yet)
static thread_local int g_cg_polls = 0;
static thread_local int g_cg_one_launch = -1;

struct CgArgs {
    const float *T;
    const double *eps;
    int n, max_iter, check, polls;
    double shift, tol;
    double *y;
    unsigned long long *slots;   // [3][n]
    double *out;                 // iterations, relative residual, 1 = done (by block 0); 1 = a block gave up
};

__global__ void cg_fill_kernel(unsigned long long *p, int64_t n, double *out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = kCgEmpty;
    if (i < 4) out[i] = 0.0;
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double cg_dpp(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROW_MASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xF, false);
    return __builtin_bit_cast(double, (long long)hi << 32 | (unsigned)lo);
}

// the sum over each row of 16 lanes, in the row's last lane
__device__ __forceinline__ double cg_row_sum(double v)
{
    v += cg_dpp<0x111, 0xF>(v);   // row_shr:1
    v += cg_dpp<0x112, 0xF>(v);   // row_shr:2
    v += cg_dpp<0x114, 0xF>(v);   // row_shr:4
    v += cg_dpp<0x118, 0xF>(v);   // row_shr:8
    return v;
}

// the sum over the wave, in its last lane (a few cycles a step; a shuffle through LDS takes about 100)
__device__ __forceinline__ double cg_wave_sum(double v)
{
    v = cg_row_sum(v);
    v += cg_dpp<0x142, 0xA>(v);   // row_bcast:15 -> rows 1, 3
    v += cg_dpp<0x143, 0xC>(v);   // row_bcast:31 -> rows 2, 3
    return v;
}

// sums of a and b over the block, the same bits in every thread (and every block); one barrier before the values are
// read and none after: callers alternate `red`
__device__ __forceinline__ void cg_sum2(double &a, double &b, double (*red)[2])
{
    a = cg_wave_sum(a);
    b = cg_wave_sum(b);
    if ((threadIdx.x & 63) == 63) {
        red[threadIdx.x >> 6][0] = a;
        red[threadIdx.x >> 6][1] = b;
    }
    __syncthreads();
    a = b = 0.0;
#pragma unroll 4
    for (int w = 0; w < kCgWaves; ++w) {
        a += red[w][0];
        b += red[w][1];
    }
}

// RW rows per wave (4 RW per block), JR column steps of 256 in registers, EM elements of the vectors per thread
template <int RW, int JR, int EM>
__global__ void __launch_bounds__(kCgThreads) sr_cg_kernel(CgArgs A)
{
    extern __shared__ __align__(16) double sm[];
    constexpr int R = kCgGroups * RW;
    const int np = max(JR, (A.n + 255) / 256) * 256;
    double *ps = sm, *ds = sm + np;                         // [np] p, zero past n; [np] 1 / (T_ii + shift)
    __shared__ double part[kCgGroups][R], red[2][kCgWaves][2];
    __shared__ int gave_up;
    const int n = A.n, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = wave % kCgGroups, rg = wave / kCgGroups, row0 = blockIdx.x * R;
    const int own = row0 + tid;                             // this thread's row of the block (tid < R)
    if (tid == 0) gave_up = 0;

    // T: rows row0 + rg RW + r, columns 256 j + 64 cg + lane; zero past n
    const int col = 64 * cg + lane, J = (n + 255) / 256;
    const float *Tr[RW];
    float t[RW][JR];
#pragma unroll
    for (int r = 0; r < RW; ++r) Tr[r] = A.T + (size_t)min(row0 + rg * RW + r, n - 1) * n;
#pragma unroll
    for (int j = 0; j < JR; ++j) {
        const int c = 256 * j + col, cc = min(c, n - 1);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const float v = Tr[r][cc];
            t[r][j] = c < n ? v : 0.0f;
        }
    }
    // right-hand side and start: r = b, z = r d, p = z
    for (int i = n + tid; i < np; i += kCgThreads) ps[i] = 0.0;
    double rv[EM];
    double se = 0.0, unused = 0.0;
#pragma unroll
    for (int e = 0; e < EM; ++e) {
        const int i = tid + kCgThreads * e;
        rv[e] = i < n ? A.eps[i] : 0.0;
        se += rv[e];
    }
    cg_sum2(se, unused, red[0]);
    const double mean = se / (double)n;
    double bb = 0.0, rz = 0.0;
#pragma unroll
    for (int e = 0; e < EM; ++e) {
        const int i = tid + kCgThreads * e;
        if (i < n) {
            const double dk = (double)A.T[(size_t)i * n + i] + A.shift, d = dk > 0.0 ? 1.0 / dk : 1.0;
            rv[e] -= mean;
            const double z = rv[e] * d;
            ds[i] = d;
            ps[i] = z;
            bb = fma(rv[e], rv[e], bb);
            rz = fma(rv[e], z, rz);
        }
    }
    cg_sum2(bb, rz, red[1]);
    double x = 0.0;                                         // of the row `own`
    double rel = 0.0;
    int k = 0;
    if (bb > 0.0) {
        rel = 1.0;
        unsigned long long *buf = A.slots, *next = A.slots + n, *prev = A.slots + 2 * (size_t)n;
        while (true) {
            __syncthreads();                                // p
            double acc[RW];
#pragma unroll
            for (int r = 0; r < RW; ++r) acc[r] = 0.0;
#pragma unroll
            for (int j = 0; j < JR; ++j) {
                const double pv = ps[256 * j + col];
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    // (t stays FP32 in its registers: widened once before the loop it would not fit them)
                    asm volatile("" : "+v"(t[r][j]));
                    acc[r] = fma((double)t[r][j], pv, acc[r]);
                }
            }
            for (int j = JR; j < J; ++j) {
                const int c = 256 * j + col;
                const double pv = ps[c];
                const int cc = min(c, n - 1);
#pragma unroll
                for (int r = 0; r < RW; ++r) acc[r] = fma((double)Tr[r][cc], pv, acc[r]);
            }
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const double s = cg_wave_sum(acc[r]);
                if (lane == 63) part[cg][rg * RW + r] = s;
            }
            __syncthreads();
            double pown = 0.0;
            if (tid < R && own < n) {
                pown = ps[own];
                double a = 0.0;
#pragma unroll
                for (int c = 0; c < kCgGroups; ++c) a += part[c][tid];
                a = fma(A.shift, pown, a);
                // the reset of `prev` of the last iteration is done before this value can be seen
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __hip_atomic_store(buf + own, __builtin_bit_cast(unsigned long long, a), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            // all n values of T p
            double ap[EM];
            {
                int spins = 0;
                bool waiting = true;
                while (waiting) {
                    unsigned long long v[EM];
#pragma unroll
                    for (int e = 0; e < EM; ++e) {
                        const int i = tid + kCgThreads * e;
                        v[e] = __hip_atomic_load(buf + min(i, n - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    waiting = false;
#pragma unroll
                    for (int e = 0; e < EM; ++e) {
                        waiting = waiting || v[e] == kCgEmpty;
                        ap[e] = __builtin_bit_cast(double, v[e]);
                    }
                    if (waiting && ++spins >= A.polls) {
                        gave_up = 1;
                        waiting = false;
                    }
                }
            }
            double pap = 0.0;
#pragma unroll
            for (int e = 0; e < EM; ++e) {
                const int i = tid + kCgThreads * e;
                if (i < n) pap = fma(ps[i], ap[e], pap);
            }
            cg_sum2(pap, unused, red[0]);
            if (gave_up) {                                  // uniform: read behind the barrier of the sum
                if (tid == 0) A.out[3] = 1.0;
                return;
            }
            if (tid < R && own < n)
                __hip_atomic_store(prev + own, kCgEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const double alpha = pap != 0.0 ? rz / pap : 0.0;
            x = fma(alpha, pown, x);
            double rz1 = 0.0, rr = 0.0;
#pragma unroll
            for (int e = 0; e < EM; ++e) {
                const int i = tid + kCgThreads * e;
                if (i < n) {
                    rv[e] = fma(-alpha, ap[e], rv[e]);
                    rz1 = fma(rv[e], rv[e] * ds[i], rz1);
                    rr = fma(rv[e], rv[e], rr);
                }
            }
            cg_sum2(rz1, rr, red[1]);
            ++k;
            if (k % A.check == 0 || k == A.max_iter) {
                rel = sqrt(rr / bb);
                if (!(rel > A.tol) || k == A.max_iter) break;   // converged, not a number, or the last iteration
            }
            const double beta = rz != 0.0 ? rz1 / rz : 0.0;
            rz = rz1;
#pragma unroll
            for (int e = 0; e < EM; ++e) {
                const int i = tid + kCgThreads * e;
                if (i < n) ps[i] = fma(beta, ps[i], rv[e] * ds[i]);
            }
            unsigned long long *was = prev;
            prev = buf;
            buf = next;
            next = was;
        }
    }
    if (tid < R && own < n) A.y[own] = x;
    if (blockIdx.x == 0 && tid == 0) {
        A.out[0] = (double)k;
        A.out[1] = rel;
        A.out[2] = 1.0;
    }
}

size_t cg_resident_bytes(int64_t n) { return 3 * sizeof(double) * (size_t)n + 64; }

// Solves in one launch and waits for it; *done = false when the launch does not apply (size, device, y in the energies'
// buffer) or gave up, with nothing that the caller's own solve would not overwrite.  ws: cg_resident_bytes(n).
nqs_status cg_resident(const float *T, const double *eloc, int64_t n, double shift, double tol, int max_iter, int check,
                       double *y, void *ws, int *iters, double *rel, bool *done, hipStream_t stream)
{
    *done = false;
    g_cg_one_launch = 0;
    // (one sample's centred energy is zero: nothing to solve)  y is written while other blocks may still read eloc only
    // if the two overlap
    if (n < 2 || n > kCgMax || (y < eloc + n && eloc < y + n)) return NQS_OK;
    // rows per wave: as many as let at most one block per CU hold all rows
    const int cus = device_cus();
    const void *kernel = nullptr;
    int RW = 0, JR = 0;
    if (n <= 512) RW = 4, JR = 2, kernel = (const void *)sr_cg_kernel<4, 2, 1>;
    else if (n <= 1024) RW = 4, JR = 4, kernel = (const void *)sr_cg_kernel<4, 4, 1>;
    else if (n <= 2048) RW = 4, JR = 8, kernel = (const void *)sr_cg_kernel<4, 8, 2>;
    else if (n <= 4096) RW = 4, JR = 16, kernel = (const void *)sr_cg_kernel<4, 16, 4>;
    else RW = 5, JR = 12, kernel = (const void *)sr_cg_kernel<5, 12, 5>;
    const int64_t blocks = (n + 4 * RW - 1) / (4 * RW);
    int dev = 0, coop = 0;
    const size_t lds = 2 * sizeof(double) * 256 * std::max<size_t>(JR, (n + 255) / 256);
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
        blocks > cus)
        return NQS_OK;
    if (lds > 60 * 1024 &&
        hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return NQS_OK;
    }
    CgArgs A;
    A.T = T;
    A.eps = eloc;
    A.n = (int)n;
    A.max_iter = max_iter;
    A.check = check;
    A.polls = g_cg_polls > 0 ? g_cg_polls : kCgPolls;
    A.shift = shift;
    A.tol = tol;
    A.y = y;
    A.slots = (unsigned long long *)ws;
    A.out = (double *)ws + 3 * n;
    hipLaunchKernelGGL(cg_fill_kernel, dim3((unsigned)((3 * n + 4 + 255) / 256)), dim3(256), 0, stream, A.slots, 3 * n, A.out);
    NQS_HIP_TRY(hipGetLastError());
    void *args[] = {&A};
    if (hipLaunchCooperativeKernel(kernel, dim3((unsigned)blocks), dim3(kCgThreads), args, (unsigned)lds, stream) !=
        hipSuccess) {
        (void)hipGetLastError();
        return NQS_OK;
    }
    double out[4] = {0.0, 0.0, 0.0, 0.0};
    NQS_HIP_TRY(hipMemcpyAsync(out, A.out, sizeof(out), hipMemcpyDeviceToHost, stream));
    NQS_HIP_TRY(hipStreamSynchronize(stream));
    if (out[2] != 1.0 || out[3] != 0.0) return NQS_OK;
    *iters = (int)out[0];
    *rel = out[1];
    *done = true;
    g_cg_one_launch = 1;
    return NQS_OK;
}

}  // namespace nqs

extern "C" int32_t nqs_probe_solve_one_launch(void) { return nqs::g_cg_one_launch; }

extern "C" void nqs_probe_solve_polls(int32_t polls) { nqs::g_cg_polls = polls > 0 ? polls : 0; }
