// Dense networks of any depth: every Metropolis step evaluates the proposed
// configurations of all chains as one batch of GEMMs on the matrix cores
// (the batched forward pass of Sec. III, one matrix product per layer).
//
// Per step (move k):
//   step      one thread per chain: the decision on move k - 1 (Delta = 2 (f' - f)
//             in FP32, accept iff log2 u < Delta / ln 2; an accepted move flips the
//             chain's spins and keeps f'; no incremental state: f is always a full
//             forward), then the draw of (i, j, u) from the chain's Philox stream
//             and whether the move changes the state (every flip, an exchange of
//             unequal spins).
//   rows      the moves that do get a row each, in chain order; 16-bit and E4M3
//             copies: their configurations as operands, +-1 with sites i, j negated
//             (exact in every format).
//   layer l   GEMM  H_l = ReLU(H_{l-1} W_l^T + b_l), rounded to the operand
//             format by the epilogue (the next product's input).
//   last      GEMM with a log-cosh epilogue: per row, the partial sums over
//             each 64-output slice are written, then added in slice order.
// The GEMM of the 16-bit and E4M3 copies is deep_frag_gemm_kernel (operands kept
// in the order of the matrix instructions); the FP32 copy runs deep_gemm_kernel:
// 128 x 128 output tile per block of 4 waves (2 x 2 v_mfma 32x32 tiles each),
// contraction steps of 128 bytes per row, operands staged through registers into
// double-buffered LDS (one barrier per step).
// Local energies use the same GEMMs on the rows (sample, connected
// configuration) of a batch of samples.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "ffnn_mc.h"
#include "internal.h"

namespace nqs {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // 16 staged bytes
typedef int i32x8 __attribute__((ext_vector_type(8)));             // 32 FP8 codes

// An OCP E4M3 code (1 sign, 4 exponent bits with bias 7, 3 mantissa bits) as a
// matrix-core operand.  Products on v_mfma_f32_32x32x64_f8f6f4 (both operands
// E4M3, unscaled), FP32 accumulation; a lane holds 32 consecutive K values.
struct Fp8 {
    uint8_t v;
};

template <>
struct Mc<Fp8> {
    static constexpr int EPL = 32;   // K elements per lane per instruction (K = 64)
    typedef i32x8 frag;
    static __device__ __forceinline__ mc_floatx16 mma(frag a, frag b, mc_floatx16 c)
    {
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
    }
};

// E4M3 code of v, 0 <= v < 464 (the scaled layer outputs never exceed 448), rounded to nearest even:
// normal values drop 20 of FP32's 23 mantissa bits (the carry of a round-up moves into the exponent),
// values below 2^-6 are multiples of the subnormal step 2^-9.
__device__ __forceinline__ uint32_t e4m3_code_nonneg(float v)
{
    const uint32_t x = __float_as_uint(v);
    const uint32_t nrm = ((x + 0x7FFFFu + ((x >> 20) & 1u)) >> 20) - (120u << 3);
    const uint32_t sub = (uint32_t)__builtin_rintf(v * 512.0f);
    return v < 0.015625f ? sub : nrm;
}

constexpr int kDT = 128;   // output tile side
constexpr int kDBytes = 128;   // contraction bytes per row per step

struct DeepGemmArgs {
    const void *A;             // activations [rows][lda] (operand format), when not from spins
    int lda;
    const int8_t *spins;       // [chains][N], when the A operand comes from spins
    const int *row_chain;      // row -> chain (or sample)
    const int *row_i;          // flipped sites of the row (-1: none)
    const int *row_j;
    int N;
    const int *nrows;          // device: number of rows
    const void *W;             // [Np][Kp] operand format
    const float *bias;         // [Np]
    int Kp, Nout, Np;
    void *out;                 // ReLU: [rows][ldo] operand format; log-cosh: float [rows][2 nct]
    int ldo;
    int nct;                   // output column tiles
    int max_row_tiles;
};

// Bit pattern of +-1 (or 0) in the operand format.
template <typename T>
__device__ __forceinline__ uint32_t deep_pm1_bits(int s)
{
    constexpr uint32_t one = sizeof(T) == 4 ? 0x3F800000u
                           : (sizeof(T) == 1 ? 0x38u : (std::is_same<T, _Float16>::value ? 0x3C00u : 0x3F80u));
    constexpr uint32_t sign = sizeof(T) == 4 ? 0x80000000u : (sizeof(T) == 1 ? 0x80u : 0x8000u);
    return s == 0 ? 0u : (one | (s < 0 ? sign : 0u));
}

// Four 16-byte staging registers of a thread (rows r, r+32, r+64, r+96).
struct Stage4 {
    u32x4 x0, x1, x2, x3;
};

// Weights -> registers: 4 rows x 16 bytes per thread (padded, always in range).
template <typename T>
__device__ __forceinline__ void deep_load_w(const DeepGemmArgs &g, int r0, int ks, Stage4 &v)
{
    constexpr int EPC = 16 / sizeof(T), BK = kDBytes / sizeof(T);
    const int tid = threadIdx.x;
    const int k0 = ks * BK + (tid & 7) * EPC;
    const u32x4 *W = reinterpret_cast<const u32x4 *>(reinterpret_cast<const T *>(g.W) + (size_t)(r0 + (tid >> 3)) * g.Kp + k0);
    const size_t step = (size_t)32 * g.Kp * sizeof(T) / 16;
    v.x0 = W[0];
    v.x1 = W[step];
    v.x2 = W[2 * step];
    v.x3 = W[3 * step];
}

// The A operand of a GEMM: activations (AM_ACT), or the chain's spins with the row's sites negated (AM_SPINS).  The
// AM_ACT path has no branch: rows past the count read a valid address and are zeroed by selects, so the compiler can
// track the loads in flight exactly (a branch around a load makes it wait for every outstanding load at the join).
constexpr int AM_ACT = 0, AM_SPINS = 2;

// Rows -> registers (rows r0 + tid / 8 + 32 q, 16 bytes of step ks each)
template <typename T, int AM>
__device__ __forceinline__ void deep_load_a(const DeepGemmArgs &g, int r0, int ks, int nrows, const int (&rc)[4],
                                            const int (&ri)[4], const int (&rj)[4], Stage4 &v)
{
    constexpr int EPC = 16 / sizeof(T), BK = kDBytes / sizeof(T);
    const int tid = threadIdx.x;
    const int k0 = ks * BK + (tid & 7) * EPC;
    auto one = [&](int q) -> u32x4 {
        const int row = r0 + (tid >> 3) + 32 * q;
        if constexpr (AM == AM_ACT) {
            const T *A = reinterpret_cast<const T *>(g.A);
            const u32x4 d = *reinterpret_cast<const u32x4 *>(A + (size_t)(row < nrows ? row : 0) * g.lda + k0);
            const bool ok = row < nrows;
            return u32x4{ok ? d.x : 0u, ok ? d.y : 0u, ok ? d.z : 0u, ok ? d.w : 0u};
        } else {
            uint32_t w0 = 0u, w1 = 0u, w2 = 0u, w3 = 0u;
            if (row < nrows) {
                const int8_t *sp = g.spins + (size_t)rc[q] * g.N;
#pragma unroll
                for (int x = 0; x < EPC; ++x) {
                    const int k = k0 + x;
                    int sv = k < g.N ? (int)sp[k] : 0;
                    if (k == ri[q] || k == rj[q]) sv = -sv;
                    const uint32_t bits = deep_pm1_bits<T>(sv);
                    const int word = sizeof(T) == 4 ? x : (sizeof(T) == 2 ? (x >> 1) : (x >> 2));
                    const uint32_t sh = sizeof(T) == 4 ? 0u : (sizeof(T) == 2 ? 16u * (x & 1) : 8u * (x & 3));
                    if (word == 0) w0 |= bits << sh;
                    else if (word == 1) w1 |= bits << sh;
                    else if (word == 2) w2 |= bits << sh;
                    else w3 |= bits << sh;
                }
            }
            return u32x4{w0, w1, w2, w3};
        }
    };
    v.x0 = one(0);
    v.x1 = one(1);
    v.x2 = one(2);
    v.x3 = one(3);
}

template <typename T>
__device__ __forceinline__ void deep_store(T *dst, const Stage4 &v)
{
    constexpr int LD = kDBytes / sizeof(T) + 16 / sizeof(T);
    constexpr int EPC = 16 / sizeof(T);
    const int tid = threadIdx.x, c = tid & 7;
    u32x4 *p = reinterpret_cast<u32x4 *>(dst + (tid >> 3) * LD + c * EPC);
    constexpr int step = 32 * LD * sizeof(T) / 16;
    p[0] = v.x0;
    p[step] = v.x1;
    p[2 * step] = v.x2;
    p[3 * step] = v.x3;
}

// A fragment of LDS
template <typename T>
__device__ __forceinline__ typename Mc<T>::frag deep_frag(const T *p)
{
    return *reinterpret_cast<const typename Mc<T>::frag *>(p);
}

template <typename T, int AM, bool LOGCOSH>
__global__ void __launch_bounds__(256, 2) deep_gemm_kernel(DeepGemmArgs g)
{
    constexpr bool SPINS = AM != AM_ACT;
    typedef typename Mc<T>::frag frag;
    constexpr int BK = kDBytes / sizeof(T);
    constexpr int LD = BK + 16 / sizeof(T);
    constexpr int EPL = Mc<T>::EPL;
    constexpr int KI = BK / (2 * EPL);            // MFMA steps per contraction step
    constexpr int TILE = kDT * LD;
    extern __shared__ __align__(16) unsigned char smem[];
    T *lds = reinterpret_cast<T *>(smem);

    const int nrows = *g.nrows;
    // The grid covers the largest row count; only `valid` tiles have work.  Block b takes tiles b, b + G,
    // b + 2G, ... (G = gridDim.x, a multiple of 8): the loads of a tile's first two contraction steps are
    // issued during the previous tile's last two, so a tile starts without waiting for memory.  Tile ids are
    // renumbered so that each XCD (blocks are dealt to the 8 XCDs round-robin) gets a contiguous range:
    // consecutive ids share a row tile, whose rows then stay in that XCD's L2.
    const int valid = ((nrows + kDT - 1) / kDT) * g.nct;
    if ((int)blockIdx.x >= valid) return;
    const int q8 = valid >> 3, r8 = valid & 7, G = gridDim.x;
    auto coords = [&](int x, int &m0, int &n0, int &ct) {
        const int xcd = x & 7, lb = xcd * q8 + min(xcd, r8) + (x >> 3);
        const int rt = lb / g.nct;
        ct = lb - rt * g.nct;
        m0 = rt * kDT;
        n0 = ct * kDT;
    };

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int l32 = lane & 31, h = lane >> 5;

    // the chain (or sample) and flipped sites of this thread's four staged rows of a tile
    auto rowinfo = [&](int m0, int (&rc)[4], int (&ri)[4], int (&rj)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            rc[q] = 0;
            ri[q] = -1;
            rj[q] = -1;
            if constexpr (SPINS) {
                const int row = m0 + (tid >> 3) + 32 * q;
                if (row < nrows) {
                    rc[q] = g.row_chain[row];
                    ri[q] = g.row_i[row];
                    rj[q] = g.row_j[row];
                }
            }
        }
    };
    int x = blockIdx.x, m0, n0, ct, m0n = 0, n0n = 0, ctn = 0;
    int rc[4], ri[4], rj[4], rcn[4], rin[4], rjn[4];
    coords(x, m0, n0, ct);
    rowinfo(m0, rc, ri, rj);
    bool has_next = x + G < valid;
    if (has_next) {
        coords(x + G, m0n, n0n, ctn);
        rowinfo(m0n, rcn, rin, rjn);
    }

    mc_floatx16 acc[2][2];
    auto zero_acc = [&]() {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
    };
    zero_acc();

    // The tile's output: ReLU rows in the operand format, or per-row log-cosh partials per 64-output slice.
    // The accumulators hold D[i = output][j = row]: lane = j + 32 ((i / 4) % 2), register = i % 4 + 4 (i / 8), so a
    // lane has row l32 of its 32-row block and outputs 8q + 4h + 0..3 (q = 0..3) of each 32-output block: four
    // consecutive outputs, stored together.  The bias of those outputs is read once, before any store.
    auto epilogue = [&](int m0, int n0, int ct) {
        float4 bq[2][4];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                bq[b][q] = *reinterpret_cast<const float4 *>(g.bias + n0 + wn + 32 * b + 8 * q + 4 * h);
        auto pre = [&](int a, int b, int q, int e) {   // the pre-activation of output 8q + 4h + e
            const float bb = e == 0 ? bq[b][q].x : (e == 1 ? bq[b][q].y : (e == 2 ? bq[b][q].z : bq[b][q].w));
            return acc[a][b][4 * q + e] + bb;
        };
        if constexpr (LOGCOSH) {
            float *part = reinterpret_cast<float *>(g.out);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                float abs_sum = 0.0f, prod = 1.0f;
                int cnt = 0;
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int col = n0 + wn + 32 * b + 8 * q + 4 * h + e;
                            if (col < g.Nout) {
                                const float v = fabsf(pre(a, b, q, e));
                                abs_sum += v;
                                prod *= 1.0f + __expf(-2.0f * v);   // 32 factors in (1, 2]
                                ++cnt;
                            }
                        }
                float sv = abs_sum + __logf(prod) - (float)cnt * kLn2f;
                sv += __shfl_xor(sv, 32, 64);
                const int row = m0 + wm + 32 * a + l32;
                if (h == 0 && row < nrows) part[(size_t)row * (2 * g.nct) + 2 * ct + (wn >> 6)] = sv;
            }
        } else {
            struct alignas(4 * sizeof(T)) Out4 {
                T v[4];
            };
            T *out = reinterpret_cast<T *>(g.out);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int row = m0 + wm + 32 * a + l32;
                if (row >= nrows) continue;
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int col0 = n0 + wn + 32 * b + 8 * q + 4 * h;
                        if (col0 >= g.ldo) continue;   // ldo is a multiple of 4: the group is whole
                        Out4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            o.v[e] = Mc<T>::from_f32(col0 + e < g.Nout ? fmaxf(pre(a, b, q, e), 0.0f) : 0.0f);
                        }
                        *reinterpret_cast<Out4 *>(out + (size_t)row * g.ldo + col0) = o;
                    }
            }
        }
    };

    // Contraction steps of all the block's tiles in sequence (ksteps >= 2 whenever a block has more than one
    // tile).  Two register stages: the loads of step v + 2 are issued before step v is computed, so each
    // global load has two steps of matrix-core work to land; across a tile boundary they are the next tile's.
    const int ksteps = g.Kp / BK;
    const int ntile = (valid - 1 - (int)blockIdx.x) / G + 1;
    const int V = ntile * ksteps;
    int ks = 0;   // step within the current tile
    // loads of step ks + d of the sequence (ksd = ks + d), without a branch: past the current tile they are
    // the next tile's; past the block's last step they read the current tile again and are never stored
    auto load = [&](int ksd, Stage4 &av, Stage4 &bv) {
        const bool nxt = ksd >= ksteps && has_next;
        int k = ksd >= ksteps ? ksd - ksteps : ksd;
        k = k < ksteps ? k : 0;
        int rca[4], ria[4], rja[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            rca[q] = nxt ? rcn[q] : rc[q];
            ria[q] = nxt ? rin[q] : ri[q];
            rja[q] = nxt ? rjn[q] : rj[q];
        }
        deep_load_a<T, AM>(g, nxt ? m0n : m0, k, nrows, rca, ria, rja, av);
        deep_load_w<T>(g, nxt ? n0n : n0, k, bv);
    };
    Stage4 a0s, b0s, a1s, b1s;
    load(0, a0s, b0s);
    load(1, a1s, b1s);
    deep_store<T>(lds, a0s);
    deep_store<T>(lds + TILE, b0s);
    __syncthreads();
    auto step = [&](int v, Stage4 &af, Stage4 &bf, const Stage4 &an, const Stage4 &bn) {
        const int cur = v & 1;
        const T *As = lds + (2 * cur) * TILE;
        const T *Bs = As + TILE;
        load(ks + 2, af, bf);
#pragma unroll
        for (int kk = 0; kk < KI; ++kk) {
            const int ko = kk * 2 * EPL + EPL * h;
            const frag a0 = deep_frag<T>(As + (wm + l32) * LD + ko);
            const frag a1 = deep_frag<T>(As + (wm + 32 + l32) * LD + ko);
            const frag b0 = deep_frag<T>(Bs + (wn + l32) * LD + ko);
            const frag b1 = deep_frag<T>(Bs + (wn + 32 + l32) * LD + ko);
            // D[i = output][j = row]
            acc[0][0] = Mc<T>::mma(b0, a0, acc[0][0]);
            acc[0][1] = Mc<T>::mma(b1, a0, acc[0][1]);
            acc[1][0] = Mc<T>::mma(b0, a1, acc[1][0]);
            acc[1][1] = Mc<T>::mma(b1, a1, acc[1][1]);
        }
        {   // after the last step this fills a buffer nothing reads
            T *nxt = lds + (2 * (cur ^ 1)) * TILE;
            deep_store<T>(nxt, an);
            deep_store<T>(nxt + TILE, bn);
        }
        __syncthreads();
        if (++ks == ksteps) {   // the tile is complete: its output, then the next tile becomes current
            epilogue(m0, n0, ct);
            zero_acc();
            ks = 0;
            x += G;
            m0 = m0n;
            n0 = n0n;
            ct = ctn;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                rc[q] = rcn[q];
                ri[q] = rin[q];
                rj[q] = rjn[q];
            }
            has_next = x + G < valid;
            if (has_next) {
                coords(x + G, m0n, n0n, ctn);
                rowinfo(m0n, rcn, rin, rjn);
            }
        }
    };
    for (int v = 0; v < V; v += 2) {
        step(v, a0s, b0s, a1s, b1s);
        if (v + 1 < V) step(v + 1, a1s, b1s, a0s, b0s);
    }
}

// ---------------------------------------------------------------------------
// 16-bit and E4M3 products on operands in matrix-instruction order (frag_index16 / frag_index8)
//
// Weights are laid out once with the copy, the spins by deep_spins_kernel, a layer's output by its epilogue (a lane
// holds four consecutive outputs of one row: half a fragment piece, so a wave's stores are whole lines); every load
// is then consecutive kilobytes.  A block of four waves takes 128 RB rows x 32 NT outputs: a wave owns 32 RB rows,
// whose operands it loads straight into registers (no other wave needs them), one contraction step (4 KB per 32 rows
// or outputs) ahead, each piece as soon as its predecessor was used; the weights are shared through double-buffered
// LDS, one barrier per step.  Tiles in sequence per block, the next tile's first loads issued in the last step.
//
// Why: with 64 x 64 outputs per wave, both operands in LDS, every product needed one LDS read, 128 bytes per clock
// of the CU, the rate of its LDS; here 64 + 16 (RB = 2, NT = 5).  The spins were expanded from bytes for each of
// the 13 column tiles, 140 vector instructions per 16 products.  400-1600-800-400 network, about 32,850 rows a
// step, BF16: layers 1 to 3 took 128, 127 and 43 us each launch, now 57, 90 and 34 us (740, 930 and 610 TFLOP/s of the
// widths asked for; bound by the LDS and operand loads of a step, which two blocks per CU overlap only in part);
// E4M3 92, 77 and 28 us, now 52, 56 and 21 us.  Layer 1 writes 105 MB and is near the rate of a copy at its end.
// Sums run over the contraction in the same order as before, so every value is the same bit for bit.
// ---------------------------------------------------------------------------
constexpr int kFragRows = 256;   // rows of the largest tile

struct DeepFragArgs {
    const u32x4 *A, *W;        // operands [32-row block][KB4][64 lanes] 16-byte pieces
    const int *nrows;          // device: number of rows
    const float *bias;         // [Np]
    int KB4;                   // pieces per block of A and W (a multiple of 4)
    int KBv;                   // contraction blocks with values
    int nbw;                   // 32-output blocks of W
    int Nout, nblk, nct;       // outputs, their 32-output blocks (what the next layer reads), column tiles
    void *out;                 // ReLU: the next layer's operands, KB4o pieces per block; log-cosh: float [rows][nslice]
    int KB4o, nslice;
    int max_row_tiles;
    float acc_scale;           // E4M3: accumulator -> pre-activation scale (weight scale x input scale)
    float next_inv;            // E4M3: 1 / scale of the next layer's input
};

template <typename T>
__device__ __forceinline__ typename Mc<T>::frag deep_frag_of(const u32x4 (&v)[sizeof(typename Mc<T>::frag) / 16])
{
    if constexpr (sizeof(typename Mc<T>::frag) == 32)
        return i32x8{(int)v[0].x, (int)v[0].y, (int)v[0].z, (int)v[0].w,
                     (int)v[1].x, (int)v[1].y, (int)v[1].z, (int)v[1].w};
    else
        return __builtin_bit_cast(typename Mc<T>::frag, v[0]);
}

template <typename T, int RB, int NT, bool LOGCOSH>
__global__ void __launch_bounds__(256, 2) deep_frag_gemm_kernel(DeepFragArgs g)
{
    typedef typename Mc<T>::frag frag;
    constexpr int P = sizeof(frag) / 16, KK = 4 / P;   // pieces per fragment, contraction blocks per step
    __shared__ u32x4 lds[2][NT * 4][64];
    const int nrows = *g.nrows;
    constexpr int kTileRows = 128 * RB;
    // tile ids are renumbered so that each XCD gets a contiguous range, whose rows stay in its L2
    const int valid = ((nrows + kTileRows - 1) / kTileRows) * g.nct, G = gridDim.x;
    if ((int)blockIdx.x >= valid) return;
    const int q8 = valid >> 3, r8 = valid & 7;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    auto coords = [&](int x, int &rb, int &nb) {   // the wave's first 32-row block, the tile's first 32-output block
        const int xcd = x & 7, lb = xcd * q8 + min(xcd, r8) + (x >> 3), rt = lb / g.nct;
        rb = (rt * 4 + wave) * RB;
        nb = (lb - rt * g.nct) * NT;
    };
    int x = blockIdx.x, rb, nb, rbn, nbn;
    coords(x, rb, nb);

    mc_floatx16 acc[RB][NT];
    u32x4 a[RB][KK][P], wr[NT];
    auto load_a = [&](int r0, int ks, int kk) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int q = 0; q < P; ++q) a[r][kk][q] = g.A[((size_t)(r0 + r) * g.KB4 + (ks * KK + kk) * P + q) * 64 + lane];
    };
    auto load_w = [&](int n0, int ks) {
#pragma unroll
        for (int b = 0; b < NT; ++b) wr[b] = g.W[((size_t)min(n0 + b, g.nbw - 1) * g.KB4 + ks * 4 + wave) * 64 + lane];
    };
    auto store_w = [&](int buf) {
#pragma unroll
        for (int b = 0; b < NT; ++b) lds[buf][b * 4 + wave][lane] = wr[b];
    };
    auto zero_acc = [&]() {
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int b = 0; b < NT; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[r][b][e] = 0.0f;
    };

    // The accumulators hold D[i = output][j = row]: lane = j + 32 ((i / 4) % 2), register = i % 4 + 4 (i / 8), so a lane
    // has row l32 of its 32-row block and outputs 8q + 4h + 0..3 (q = 0..3) of each 32-output block.
    auto epilogue = [&]() {
        auto pre = [&](int r, int b, int q, int e, const float4 &bq) {
            const float bb = e == 0 ? bq.x : (e == 1 ? bq.y : (e == 2 ? bq.z : bq.w));
            return std::is_same<T, Fp8>::value ? fmaf(acc[r][b][4 * q + e], g.acc_scale, bb) : acc[r][b][4 * q + e] + bb;
        };
        if constexpr (LOGCOSH) {
            // per row, the partial sums over each 64-output slice
            static_assert(NT % 2 == 0, "whole slices");
            float *part = reinterpret_cast<float *>(g.out);
#pragma unroll
            for (int sl = 0; sl < NT / 2; ++sl) {
                if (nb + 2 * sl >= 2 * g.nslice) break;
                float4 bq[2][4];
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        bq[b][q] = *reinterpret_cast<const float4 *>(g.bias + (nb + 2 * sl + b) * 32 + 8 * q + 4 * h);
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    float abs_sum = 0.0f, prod = 1.0f;
                    int cnt = 0;
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if ((nb + 2 * sl + b) * 32 + 8 * q + 4 * h + e < g.Nout) {
                                    const float v = fabsf(pre(r, 2 * sl + b, q, e, bq[b][q]));
                                    abs_sum += v;
                                    prod *= 1.0f + __expf(-2.0f * v);   // 32 factors in (1, 2]
                                    ++cnt;
                                }
                    float sv = abs_sum + __logf(prod) - (float)cnt * kLn2f;
                    sv += __shfl_xor(sv, 32, 64);
                    const int row = (rb + r) * 32 + l32;
                    if (h == 0 && row < nrows) part[(size_t)row * g.nslice + (nb >> 1) + sl] = sv;
                }
            }
        } else {
            // rows past the last lie within the buffer (whole tiles) and are never used
            unsigned char *out = reinterpret_cast<unsigned char *>(g.out);
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                if (nb + b >= g.nblk) break;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = (nb + b) * 32 + 8 * q + 4 * h;
                    const float4 bq = *reinterpret_cast<const float4 *>(g.bias + col);
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        struct alignas(4 * sizeof(T)) {
                            T v[4];
                        } o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float v = col + e < g.Nout ? fmaxf(pre(r, b, q, e, bq), 0.0f) : 0.0f;
                            if constexpr (std::is_same<T, Fp8>::value)
                                // the next layer's input: ReLU(z) / s_next as an E4M3 code (s_next a power of two)
                                o.v[e] = Fp8{(uint8_t)e4m3_code_nonneg(v * g.next_inv)};
                            else
                                o.v[e] = Mc<T>::from_f32(v);
                        }
                        size_t piece;
                        if constexpr (P == 2)
                            piece = ((size_t)(rb + r) * g.KB4o + (col >> 6) * 2 + ((col >> 4) & 1)) * 64 + ((col >> 5) & 1) * 32;
                        else
                            piece = ((size_t)(rb + r) * g.KB4o + (col >> 4)) * 64 + ((col >> 3) & 1) * 32;
                        constexpr int kPer = 16 / sizeof(T);   // values per piece
                        *reinterpret_cast<decltype(o) *>(out + (piece + l32) * 16 + (col % kPer) * sizeof(T)) = o;
                    }
                }
            }
        }
    };

    const int KS = (g.KBv + KK - 1) / KK, rem = g.KBv - (KS - 1) * KK;   // steps, blocks of the last one
    load_w(nb, 0);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) load_a(rb, 0, kk);
    store_w(0);
    zero_acc();
    __syncthreads();
    int cur = 0;
    // one step: products of step ks; the loads of the step that follows (row block rf, output block nf, step kf)
    auto step = [&](auto last, int rf, int nf, int kf) {
        load_w(nf, kf);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            if (!decltype(last)::value || kk < rem) {
                frag av[RB];
#pragma unroll
                for (int r = 0; r < RB; ++r) av[r] = deep_frag_of<T>(a[r][kk]);
#pragma unroll
                for (int b = 0; b < NT; ++b) {
                    u32x4 wv[P];
#pragma unroll
                    for (int q = 0; q < P; ++q) wv[q] = lds[cur][b * 4 + kk * P + q][lane];
                    const frag w = deep_frag_of<T>(wv);
                    // D[i = output][j = row]
#pragma unroll
                    for (int r = 0; r < RB; ++r) acc[r][b] = Mc<T>::mma(w, av[r], acc[r][b]);
                }
            }
            load_a(rf, kf, kk);
        }
        store_w(cur ^ 1);
        __syncthreads();
        cur ^= 1;
    };
    while (true) {
        for (int ks = 0; ks + 1 < KS; ++ks) step(std::false_type{}, rb, nb, ks + 1);
        const bool more = x + G < valid;
        rbn = rb;
        nbn = nb;
        if (more) coords(x + G, rbn, nbn);
        step(std::true_type{}, rbn, nbn, 0);
        epilogue();
        if (!more) break;
        zero_acc();
        x += G;
        rb = rbn;
        nb = nbn;
    }
}

// Piece u of a first-layer operand row: 16 bytes, that is 8 or 16 spins, of lane half u % 2.
template <typename T>
struct SpinPiece {
    static constexpr int EPC = 16 / sizeof(T);        // spins
    static constexpr int P = sizeof(typename Mc<T>::frag) / 16;
    typedef typename std::conditional<EPC == 16, unsigned __int128, uint64_t>::type raw_t;
    static __device__ __forceinline__ int first(int u)
    {
        const int pc = u >> 1, h = u & 1;
        return P == 2 ? (pc >> 1) * 64 + 32 * h + 16 * (pc & 1) : pc * 16 + 8 * h;
    }
    // the spins from the piece's first on, or the last EPC of the row where it ends past N (any bytes where N < EPC)
    static __device__ __forceinline__ raw_t load(const int8_t *sp, int N, int u)
    {
        raw_t raw = 0;
        if (N >= EPC) {
            __builtin_memcpy(&raw, sp + min(first(u), N - EPC), EPC);
        } else {
            for (int e = 0; e < N; ++e) raw |= (raw_t)(uint8_t)sp[e] << (8 * e);
        }
        return raw;
    }
    // the operand of row `row`, sites fi and fj negated
    static __device__ __forceinline__ void store(raw_t raw, int N, int u, int fi, int fj, int row, int KB4, u32x4 *X)
    {
        const int k0 = first(u), over = k0 + EPC - N;   // spins of the piece past N
        if (N >= EPC && over > 0) raw = over < EPC ? raw >> (8 * over) : (raw_t)0;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            const int k = k0 + e, sv = (int8_t)(uint8_t)(raw >> (8 * e));
            const int v = k >= N ? 0 : k == fi || k == fj ? -sv : sv;
            w[e * (int)sizeof(T) / 4] |= deep_pm1_bits<T>(v) << (8 * ((e * (int)sizeof(T)) & 3));
        }
        X[((size_t)(row >> 5) * KB4 + (u >> 1)) * 64 + (u & 1) * 32 + (row & 31)] = u32x4{w[0], w[1], w[2], w[3]};
    }
};
// Pieces loaded before the first is stored: the stores could alias the spins, so the compiler waits for the loads there.
constexpr int kPieceBatch = 4;

// The rows' configurations as first-layer operands (the sampler's proposals write their own)
template <typename T>
__global__ void __launch_bounds__(256) deep_spins_kernel(const int8_t *__restrict__ spins, const int *__restrict__ nrows,
                                                         const int *__restrict__ row_chain,
                                                         const int *__restrict__ row_i, const int *__restrict__ row_j,
                                                         int N, int KB4, int KBv, u32x4 *__restrict__ out)
{
    typedef SpinPiece<T> SP;
    const int row = blockIdx.x * 32 + (threadIdx.x & 31);
    if (row >= *nrows) return;
    const int8_t *sp = spins + (size_t)row_chain[row] * N;
    const int fi = row_i[row], fj = row_j[row], U = KBv * SP::P * 2;
    for (int u0 = threadIdx.x >> 5; u0 < U; u0 += 8 * kPieceBatch) {
        typename SP::raw_t raw[kPieceBatch];
#pragma unroll
        for (int q = 0; q < kPieceBatch; ++q) raw[q] = SP::load(sp, N, min(u0 + 8 * q, U - 1));
#pragma unroll
        for (int q = 0; q < kPieceBatch; ++q)
            if (u0 + 8 * q < U) SP::store(raw[q], N, u0 + 8 * q, fi, fj, row, KB4, out);
    }
}

// ---------------------------------------------------------------------------
// Sampler steps
// ---------------------------------------------------------------------------
struct DeepStepArgs {
    int8_t *state;            // [C][N] live chain states
    int64_t C;
    int N, move;
    uint64_t seed, step_offset;
    uint32_t inst, chain_id_offset;
    int *counter;             // rows of the step
    int *row_chain, *row_i, *row_j;   // FP32 copy: the rows' chains and sites
    int *prop_i, *prop_j;     // [C] sites of the chain's current proposal
    uint32_t *ubits;          // [C] u bits of the chain's current proposal
    unsigned long long *moves;   // [C / 64] chains whose current proposal changes the state, a bit each
    uint8_t *count;           // [C / 64] their number (whole pieces of 16)
    int *base;                // [C / 64] row of the first of them
    float *fcur;              // [C] log|psi| of the current state
    const float *part;        // [rows][npart]
    int npart;
    unsigned long long *acc;  // [C]
    int64_t total;            // proposals per chain in this call
    const int64_t *kbase;     // device: index of the current sweep's first proposal (graph replays), or NULL
    int n_traced;
    int32_t *tr_site;
    uint32_t *tr_ubits;
    float *tr_delta;
    uint8_t *tr_acc;
};

// One wave per 64 chains: the decision on proposal k - 1 (decide), then proposal k (propose).  A chain's state is final
// once its own decision is made, so both fit one launch; every load but the ones of a decision's partial sums and spins
// starts at once (the new proposal's spins are read before the decided move is written and corrected for it).
__global__ void __launch_bounds__(64) deep_step_kernel(DeepStepArgs a, int64_t kk, int decide, int propose)
{
    const int lane = threadIdx.x;
    const int64_t c = blockIdx.x * (int64_t)64 + lane, k = (a.kbase ? *a.kbase : 0) + kk;
    const bool in = c < a.C;
    const int64_t cc = in ? c : a.C - 1;
    int8_t *s = a.state + cc * a.N;
    int i = 0, j = -1, si = 0, sj = 0;
    uint32_t ub = 0;
    if (propose) {
        const uint64_t step = a.step_offset + (uint64_t)k;
        const uint32_t gid = a.chain_id_offset + (uint32_t)cc;
        const Block4 rb = philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), gid, a.inst << 8, (uint32_t)a.seed,
                                        (uint32_t)(a.seed >> 32));
        i = index_from_word(rb.r0, a.N);
        if (a.move == 1) {
            j = index_from_word(rb.r1, a.N - 1);
            j += (j >= i) ? 1 : 0;
        }
        si = s[i];
        sj = s[j < 0 ? i : j];
        ub = rb.r2 >> 8;
    }
    unsigned long long n_acc = a.acc[cc];
    if (decide) {
        const unsigned long long mv = a.moves[blockIdx.x];
        const int pi = a.prop_i[cc], pj = a.prop_j[cc];
        const uint32_t pub = a.ubits[cc];
        const float f = a.fcur[cc];
        if (in && ((mv >> lane) & 1)) {
            const float *part = a.part + (size_t)(a.base[blockIdx.x] + __popcll(mv & ((1ull << lane) - 1ull))) * a.npart;
            const int vi = s[pi], vj = s[pj < 0 ? pi : pj];
            float fnew = 0.0f;
            for (int p = 0; p < a.npart; p += 4) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = part[min(p + e, a.npart - 1)];
#pragma unroll
                for (int e = 0; e < 4; ++e) fnew = p + e < a.npart ? fnew + v[e] : fnew;
            }
            const float d2 = 2.0f * (fnew - f) / kLn2f;
            const float l2u = __builtin_amdgcn_logf((float)pub * 5.9604644775390625e-8f);
            const bool accept = l2u < d2;   // NaN rejects
            if (accept) {
                s[pi] = (int8_t)-vi;
                if (pj >= 0) s[pj] = (int8_t)-vj;
                a.fcur[c] = fnew;
                ++n_acc;
                if (i == pi || i == pj) si = -si;
                if (j == pi || j == pj) sj = -sj;   // only used where j >= 0
            }
            if (c < a.n_traced) {
                const size_t idx = (size_t)c * (size_t)a.total + (size_t)(k - 1);
                a.tr_delta[idx] = d2 * kLn2f;
                a.tr_acc[idx] = accept ? 1 : 0;
            }
        }
    }
    if (propose) {
        const bool eff = in && (j < 0 || si != sj);
        const unsigned long long bal = __ballot(eff);
        if (lane == 0) {
            a.moves[blockIdx.x] = bal;
            a.count[blockIdx.x] = (uint8_t)__popcll(bal);
        }
        if (in) {
            a.prop_i[c] = i;
            a.prop_j[c] = j;
            a.ubits[c] = ub;
            if (!eff) ++n_acc;   // a move that changes nothing is accepted
            if (c < a.n_traced) {
                const size_t idx = (size_t)c * (size_t)a.total + (size_t)k;
                a.tr_site[idx] = i | ((j < 0 ? 0xFFFF : j) << 16);
                a.tr_ubits[idx] = ub;
                if (!eff) {
                    a.tr_delta[idx] = 0.0f;
                    a.tr_acc[idx] = 1;
                }
            }
        }
    }
    if (in) a.acc[c] = n_acc;
}

// The rows of the step: the proposals that change the state, in the order of their chains (64 per block).  Each block
// adds up the counts before its own (one byte per 64 chains, so 4 KB of them per 262,144 chains), and, unless T is
// float, writes its rows' configurations as first-layer operands (KB4 pieces per 32 rows, KBv contraction blocks).
// Bound by the latency of three dependent loads below some 10,000 chains, then by the 2 N + N bytes a row.  With an
// atomic count per wave in the proposals (12.7 ns each, one word) and the operands expanded by every block of the first
// layer's product, proposal and decision took 21 us at 65,536 chains of 400 sites and 8.7 us at 8,000; step and rows take
// 20 and 13.3 us and include the operands (a launch of their own: 10 us).
template <typename T>
__global__ void __launch_bounds__(256) deep_rows_kernel(DeepStepArgs a, int KB4, int KBv, u32x4 *X)
{
    __shared__ int l_chain[64], l_i[64], l_j[64], l_sum[4];
    const int tid = threadIdx.x;
    const int64_t blk = blockIdx.x;
    const unsigned long long bal = a.moves[blk];
    const int m = __popcll(bal);
    uint32_t before = 0;
    for (int64_t q = tid; q * 16 < blk; q += 256) {
        const u32x4 v = reinterpret_cast<const u32x4 *>(a.count)[q];
        const int64_t n = blk - q * 16;   // counts of the piece that come before
        auto part = [&](uint32_t x, int w) { return n >= 4 * w + 4 ? x : n > 4 * w ? x & ((1u << (8 * (n - 4 * w))) - 1u) : 0u; };
        before = __builtin_amdgcn_sad_u8(part(v.x, 0), 0u, before);
        before = __builtin_amdgcn_sad_u8(part(v.y, 1), 0u, before);
        before = __builtin_amdgcn_sad_u8(part(v.z, 2), 0u, before);
        before = __builtin_amdgcn_sad_u8(part(v.w, 3), 0u, before);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
    if ((tid & 63) == 0) l_sum[tid >> 6] = (int)before;
    if (tid < 64 && ((bal >> tid) & 1)) {
        const int at = __popcll(bal & ((1ull << tid) - 1ull));
        const int64_t c = blk * 64 + tid;
        l_chain[at] = (int)c;
        l_i[at] = a.prop_i[c];
        l_j[at] = a.prop_j[c];
    }
    __syncthreads();
    const int base = l_sum[0] + l_sum[1] + l_sum[2] + l_sum[3];
    if (tid == 0) {
        a.base[blk] = base;
        if (blk + 1 == gridDim.x) *a.counter = base + m;
    }
    if constexpr (std::is_same<T, float>::value) {
        if (tid < m) {
            a.row_chain[base + tid] = l_chain[tid];
            a.row_i[base + tid] = l_i[tid];
            a.row_j[base + tid] = l_j[tid];
        }
    } else {
        // item u m + r: piece u of row r, so that consecutive lanes store consecutive rows' pieces
        typedef SpinPiece<T> SP;
        const int items = KBv * SP::P * 2 * m;
        const uint32_t inv = m > 1 ? 0xFFFFFFFFu / (uint32_t)m + 1u : 0u;   // it / m = umulhi(it, inv): it < 2^26, m <= 64
        for (int i0 = tid; i0 < items; i0 += 256 * kPieceBatch) {
            typename SP::raw_t raw[kPieceBatch];
            int u[kPieceBatch], r[kPieceBatch];
#pragma unroll
            for (int q = 0; q < kPieceBatch; ++q) {
                const int it = min(i0 + 256 * q, items - 1);
                u[q] = m > 1 ? (int)__umulhi((uint32_t)it, inv) : it;
                r[q] = it - u[q] * m;
                raw[q] = SP::load(a.state + (size_t)l_chain[r[q]] * a.N, a.N, u[q]);
            }
#pragma unroll
            for (int q = 0; q < kPieceBatch; ++q)
                if (i0 + 256 * q < items) SP::store(raw[q], a.N, u[q], l_i[r[q]], l_j[r[q]], base + r[q], KB4, X);
        }
    }
}

// rows = all chains, nothing flipped (the initial forward pass)
__global__ void deep_rows_all_kernel(int64_t C, int *counter, int *row_chain, int *row_i, int *row_j)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c == 0) {
        counter[0] = (int)C;
    }
    if (c >= C) return;
    row_chain[c] = (int)c;
    row_i[c] = -1;
    row_j[c] = -1;
}

__global__ void deep_set_f_kernel(int64_t C, const float *part, int npart, float *fcur, unsigned long long *acc)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= C) return;
    float f = 0.0f;
    for (int p = 0; p < npart; ++p) f += part[(size_t)c * npart + p];
    fcur[c] = f;
    acc[c] = 0ull;
}

__global__ void deep_emit_kernel(const int8_t *state, int64_t C, int N, const float *fcur, int8_t *samples,
                                 float *logpsi)
{
    const int64_t n = C * N;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        if (samples) samples[p] = state[p];
        if (logpsi && p < C) logpsi[p] = fcur[p];
    }
}

// graph replays: the emit of the sweep that starts at proposal *kbase, then the advance to the next sweep
__global__ void deep_emit_sweep_kernel(const int8_t *state, int64_t C, int N, const float *fcur, int8_t *samples,
                                       float *logpsi, const int64_t *kbase, int sweep_size, int n_burnin, int n_sweeps)
{
    const int64_t out = *kbase / sweep_size - n_burnin;
    if (out < 0 || out >= n_sweeps) return;
    const int64_t n = C * N;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        if (samples) samples[(size_t)out * n + p] = state[p];
        if (logpsi && p < C) logpsi[(size_t)out * C + p] = fcur[p];
    }
}

__global__ void deep_set_i64_kernel(int64_t *p, int64_t v, int64_t add)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *p = add ? *p + add : v;
}

__global__ void deep_copy_acc_kernel(const unsigned long long *acc, int64_t C, uint64_t *out)
{
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c < C) out[c] = acc[c];
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
template <typename T, int AM, bool LOGCOSH>
static void deep_gemm_launch(const DeepGemmArgs &g, hipStream_t s)
{
    constexpr size_t lds = 4 * sizeof(T) * kDT * (kDBytes / sizeof(T) + 16 / sizeof(T));
    allow_lds(deep_gemm_kernel<T, AM, LOGCOSH>, lds);
    // persistent blocks (two per CU, a multiple of 8 for the XCD renumbering) when a tile has at least two
    // contraction steps; otherwise one block per tile
    int blocks = g.max_row_tiles * g.nct;
    if (g.Kp / (kDBytes / (int)sizeof(T)) >= 2) blocks = std::min(blocks, 2 * device_cus());
    hipLaunchKernelGGL((deep_gemm_kernel<T, AM, LOGCOSH>), dim3(blocks), dim3(256), lds, s, g);
}

template <typename T, int RB, int NT, bool LOGCOSH>
static void deep_frag_launch(DeepFragArgs &g, int64_t cap, hipStream_t s)
{
    g.nct = (g.nblk + NT - 1) / NT;
    const int64_t tiles = (cap + 128 * RB - 1) / (128 * RB) * g.nct;
    // persistent blocks, a multiple of 8 for the XCD renumbering
    const int64_t blocks = std::min<int64_t>((tiles + 7) / 8 * 8, (RB == 2 ? 2 : 4) * (int64_t)device_cus());
    hipLaunchKernelGGL((deep_frag_gemm_kernel<T, RB, NT, LOGCOSH>), dim3((unsigned)blocks), dim3(256), 0, s, g);
}

// Scratch of one forward pass over up to `cap` rows.
struct DeepBuffers {
    int *counter, *row_chain, *row_i, *row_j;
    void *H[2];
    float *part;
    int64_t npart;
};
// (its bytes are part of the sweep graph's signature: no padding, which would differ from call to call)
static_assert(std::has_unique_object_representations_v<DeepBuffers>, "no padding");

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// operand columns of the layer inputs (the fragment path keeps the spins as operands too), and the rows, whole
// blocks of kFragRows there
static int deep_max_k(const FfnnDev &f, int esize)
{
    int maxK = 64;
    for (int l = esize == 4 ? 1 : 0; l < f.n_layers; ++l) maxK = std::max(maxK, f.Kp[l]);
    return maxK;
}
static int64_t deep_rows(int64_t cap, int esize)
{
    return esize == 4 ? cap : (cap + kFragRows - 1) / kFragRows * kFragRows;
}

// partial log-cosh sums per row: 64-output slices
static int deep_npart(const FfnnDev &f, int esize)
{
    return esize == 4 ? 2 * (f.Np[f.n_layers - 1] / kDT) : (f.widths[f.n_layers] + 63) / 64;
}

static size_t deep_buffer_bytes(const FfnnDev &f, int64_t cap, int esize)
{
    const int npart = deep_npart(f, esize);
    return al256(sizeof(int) * 2) + 3 * al256(sizeof(int) * cap) +
           2 * al256((size_t)esize * deep_rows(cap, esize) * deep_max_k(f, esize)) + al256(sizeof(float) * cap * npart);
}

static DeepBuffers deep_carve(const FfnnDev &f, int64_t cap, int esize, char *base)
{
    DeepBuffers b;
    b.npart = deep_npart(f, esize);
    auto carve = [&](size_t sz) {
        char *p = base;
        base += al256(sz);
        return p;
    };
    b.counter = (int *)carve(sizeof(int) * 2);
    b.row_chain = (int *)carve(sizeof(int) * cap);
    b.row_i = (int *)carve(sizeof(int) * cap);
    b.row_j = (int *)carve(sizeof(int) * cap);
    const size_t hb = (size_t)esize * deep_rows(cap, esize) * deep_max_k(f, esize);
    b.H[0] = carve(hb);
    b.H[1] = carve(hb);
    b.part = (float *)carve(sizeof(float) * cap * b.npart);
    return b;
}

// One forward pass of the rows listed in b on operands in matrix-instruction order (about `expect` of them, which
// only chooses the tiles); spins NULL: the first layer's operands are there.
template <typename T>
static void deep_frag_forward(const FfnnDev &f, const DeepBuffers &b, const int8_t *spins, int64_t cap, int64_t expect,
                              hipStream_t s)
{
    constexpr int KM = 2 * Mc<T>::EPL, P = sizeof(typename Mc<T>::frag) / 16;
    const int L = f.n_layers, N = f.widths[0];
    if (spins)
        hipLaunchKernelGGL(deep_spins_kernel<T>, dim3((unsigned)((cap + 31) / 32)), dim3(256), 0, s, spins, b.counter,
                           b.row_chain, b.row_i, b.row_j, N, f.Kp[0] / KM * P, (N + KM - 1) / KM, (u32x4 *)b.H[1]);
    for (int l = 0; l < L; ++l) {
        const bool last = l == L - 1;
        DeepFragArgs g;
        g.A = (const u32x4 *)b.H[(l + 1) & 1];
        g.W = (const u32x4 *)f.Wd[l];
        g.nrows = b.counter;
        g.bias = f.bd[l];
        g.KB4 = f.Kp[l] / KM * P;
        g.KBv = (f.widths[l] + KM - 1) / KM;
        g.nbw = f.Np[l] / 32;
        g.Nout = f.widths[l + 1];
        g.nblk = last || KM == 64 ? 2 * ((g.Nout + 63) / 64) : (g.Nout + 31) / 32;
        g.out = last ? (void *)b.part : b.H[l & 1];
        g.KB4o = last ? 0 : f.Kp[l + 1] / KM * P;
        g.nslice = b.npart;
        g.acc_scale = f.acc_scale[l];
        g.next_inv = f.next_inv[l];
        // The tile whose busiest CU is done first.  `pair`: two 256 x 32 NT tiles side by side on a CU, 0.31 us per 64
        // of the contraction (measured 0.99, 1.32, 1.67 and 1.91 us for NT = 2 to 5 on 1600 x 800 weights); one tile
        // alone takes 0.7 of that; 128 x 64 tiles, four side by side, 0.94 of the unit each, fewer 1.06 + 0.58 t.  With
        // 1600 x 800 weights the choice is 128 x 64 below 5,500 rows (4,000: 21.4 us, 256 x 64 24.6), 256 x 64 at 8,200
        // (29.6; 128 x 64 33.4, 256 x 128 34.7), 256 x 96 at 12,000 (36.6; 256 x 128 43.7), 256 x 128 at 16,400
        // (46.3; 256 x 64 51.7, 256 x 160 51.5) and 256 x 160 at 32,800 (84.7; 256 x 128 89.8).  The constants are those of
        // 1600 x 800 weights in BF16.  Elsewhere, steps of 500 to 65,536 rows of the networks 64-250-130-70, 100-400-200-100,
        // 256-1024-512-256, 400-1600-800-400 and 144-2000-300-1500 take from 0.93 to 1.04 times the best step with one tile
        // for all layers in 16 bits, to 1.07 times in E4M3 (worst: 6,000 rows of the last, 51.5 us, 128 x 64 48.0).
        const int64_t cus = device_cus();
        auto tiles = [&](int RB, int NT) {   // of the busiest CU
            return (double)(((expect + 128 * RB - 1) / (128 * RB) * ((g.nblk + NT - 1) / NT) + cus - 1) / cus);
        };
        auto cost = [&](int NT, double pair) { return (tiles(2, NT) + 0.4 * std::fmod(tiles(2, NT), 2)) * 0.5 * pair; };
        const double t = tiles(1, 2), c1 = std::max(0.94 * t, 1.06 + 0.58 * t);
        const double c2 = cost(2, 3.2), c3 = cost(3, 4.25), c4 = cost(4, 5.4), c5 = cost(5, 6.15);
        if (last) {
            if (c1 <= std::min(c2, c4)) deep_frag_launch<T, 1, 2, true>(g, cap, s);
            else if (c2 <= c4) deep_frag_launch<T, 2, 2, true>(g, cap, s);
            else deep_frag_launch<T, 2, 4, true>(g, cap, s);
        } else {
            const double c = std::min(std::min(std::min(c1, c2), std::min(c3, c4)), c5);
            if (c == c1) deep_frag_launch<T, 1, 2, false>(g, cap, s);
            else if (c == c2) deep_frag_launch<T, 2, 2, false>(g, cap, s);
            else if (c == c3) deep_frag_launch<T, 2, 3, false>(g, cap, s);
            else if (c == c4) deep_frag_launch<T, 2, 4, false>(g, cap, s);
            else deep_frag_launch<T, 2, 5, false>(g, cap, s);
        }
    }
}

// One forward pass of the rows listed in b (count on the device), spins from `spins`.
static void deep_forward(int dtype, const FfnnDev &f, const DeepBuffers &b, const int8_t *spins, int64_t cap,
                         int64_t expect, bool spins_ready, hipStream_t s)
{
    const int L = f.n_layers;
    if (dtype == NQS_BF16) return deep_frag_forward<__bf16>(f, b, spins_ready ? nullptr : spins, cap, expect, s);
    if (dtype == NQS_F16) return deep_frag_forward<_Float16>(f, b, spins_ready ? nullptr : spins, cap, expect, s);
    if (dtype == NQS_FP8_E4M3) return deep_frag_forward<Fp8>(f, b, spins_ready ? nullptr : spins, cap, expect, s);
    DeepGemmArgs g;
    g.spins = spins;
    g.row_chain = b.row_chain;
    g.row_i = b.row_i;
    g.row_j = b.row_j;
    g.N = f.widths[0];
    g.nrows = b.counter;
    g.max_row_tiles = (int)((cap + kDT - 1) / kDT);
    for (int l = 0; l < L; ++l) {
        const bool last = l == L - 1;
        g.A = l == 0 ? nullptr : b.H[(l - 1) & 1];
        g.lda = f.Kp[l];
        g.W = f.Wd[l];
        g.bias = f.bd[l];
        g.Kp = f.Kp[l];
        g.Nout = f.widths[l + 1];
        g.Np = f.Np[l];
        g.nct = f.Np[l] / kDT;
        g.out = last ? (void *)b.part : b.H[l & 1];
        g.ldo = last ? 0 : f.Kp[l + 1];
        if (l == 0) last ? deep_gemm_launch<float, AM_SPINS, true>(g, s) : deep_gemm_launch<float, AM_SPINS, false>(g, s);
        else last ? deep_gemm_launch<float, AM_ACT, true>(g, s) : deep_gemm_launch<float, AM_ACT, false>(g, s);
    }
}

nqs_status deep_sample(nqs_model *m, const nqs_sample_cfg &cfg, int8_t *chain_state, int8_t *samples, float *logpsi,
                       uint64_t *n_accepted, const nqs_trace *trace, hipStream_t stream)
{
    const FfnnDev &f = m->copies[cfg.dtype].ffnn;
    const int N = f.widths[0];
    const int64_t C = cfg.n_chains;
    const int esize = cfg.dtype == NQS_F32 ? 4 : (cfg.dtype == NQS_FP8_E4M3 ? 1 : 2);
    if (C > INT32_MAX / 2) return set_error(NQS_EINVAL, "too many chains");
    // scratch: forward buffers + per-chain state
    const size_t fwd = deep_buffer_bytes(f, C, esize);
    const int64_t nw = (C + 63) / 64;
    const size_t per_chain = 3 * al256(sizeof(int) * C) + al256(sizeof(float) * C) + al256(sizeof(unsigned long long) * C) +
                             al256(sizeof(unsigned long long) * nw) + al256((size_t)(nw + 15) / 16 * 16) +
                             al256(sizeof(int) * nw) + al256(sizeof(int64_t));
    char *ws = (char *)workspace(fwd + per_chain, stream);
    if (!ws) return set_error(NQS_ENOMEM, "workspace allocation failed");
    DeepBuffers b = deep_carve(f, C, esize, ws);
    char *pc = ws + fwd;
    auto carve = [&](size_t bytes) {
        char *p = pc;
        pc += al256(bytes);
        return (void *)p;
    };
    DeepStepArgs a = {};
    a.prop_i = (int *)carve(sizeof(int) * C);
    a.prop_j = (int *)carve(sizeof(int) * C);
    a.ubits = (uint32_t *)carve(sizeof(uint32_t) * C);
    float *fcur = (float *)carve(sizeof(float) * C);
    unsigned long long *acc = (unsigned long long *)carve(sizeof(unsigned long long) * C);
    a.moves = (unsigned long long *)carve(sizeof(unsigned long long) * nw);
    a.count = (uint8_t *)carve((size_t)(nw + 15) / 16 * 16);
    a.base = (int *)carve(sizeof(int) * nw);
    int64_t *kbase = (int64_t *)carve(sizeof(int64_t));

    if (cfg.init_chains) {
        nqs_status st = launch_init_chains(chain_state, C, N, cfg.move, cfg.seed, cfg.instance_id, cfg.chain_id_offset,
                                           stream);
        if (st != NQS_OK) return st;
    }
    const unsigned cb = (unsigned)((C + 255) / 256);
    // f of the start states
    hipLaunchKernelGGL(deep_rows_all_kernel, dim3(cb), dim3(256), 0, stream, C, b.counter, b.row_chain, b.row_i, b.row_j);
    deep_forward(cfg.dtype, f, b, chain_state, C, C, false, stream);
    hipLaunchKernelGGL(deep_set_f_kernel, dim3(cb), dim3(256), 0, stream, C, b.part, b.npart, fcur, acc);
    NQS_HIP_TRY(hipGetLastError());

    a.state = chain_state;
    a.C = C;
    a.N = N;
    a.move = cfg.move;
    a.seed = cfg.seed;
    a.step_offset = cfg.step_offset;
    a.inst = cfg.instance_id;
    a.chain_id_offset = (uint32_t)cfg.chain_id_offset;
    a.counter = b.counter;
    a.row_chain = b.row_chain;
    a.row_i = b.row_i;
    a.row_j = b.row_j;
    a.fcur = fcur;
    a.part = b.part;
    a.npart = b.npart;
    a.acc = acc;
    const int sw = cfg.sweep_size > 0 ? cfg.sweep_size : N;
    a.total = (int64_t)(cfg.n_burnin + cfg.n_sweeps) * sw;
    const bool tr = trace && trace->n_chains_traced > 0;
    a.n_traced = tr ? trace->n_chains_traced : 0;
    a.tr_site = tr ? trace->site : nullptr;
    a.tr_ubits = tr ? trace->ubits : nullptr;
    a.tr_delta = tr ? trace->delta : nullptr;
    a.tr_acc = tr ? trace->accepted : nullptr;
    a.kbase = nullptr;
    // half of the exchanges swap unequal spins
    const int64_t expect = cfg.move == NQS_MOVE_EXCHANGE ? std::max<int64_t>(1, C / 2 * N / (N - 1)) : C;
    // the decision on proposal k - 1, unless k is a sweep's first, and proposal k with its forward pass; the decision on a
    // sweep's last proposal
    auto decide = [&](int64_t k, int dec, int pro, hipStream_t s) {
        hipLaunchKernelGGL(deep_step_kernel, dim3((unsigned)nw), dim3(64), 0, s, a, k, dec, pro);
    };
    auto step = [&](int64_t k, int first, hipStream_t s) {
        decide(k, !first, 1, s);
        auto rows = [&](auto kernel, int KM, int P) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)nw), dim3(256), 0, s, a, f.Kp[0] / KM * P, (N + KM - 1) / KM,
                               (u32x4 *)b.H[1]);
        };
        if (cfg.dtype == NQS_BF16) rows(deep_rows_kernel<__bf16>, 16, 1);
        else if (cfg.dtype == NQS_F16) rows(deep_rows_kernel<_Float16>, 16, 1);
        else if (cfg.dtype == NQS_FP8_E4M3) rows(deep_rows_kernel<Fp8>, 64, 2);
        else rows(deep_rows_kernel<float>, 16, 1);
        deep_forward(cfg.dtype, f, b, chain_state, C, expect, true, s);
    };

    // Two or more sweeps: capture one sweep's launches (proposal, forward pass, decision for each
    // of its proposals, then the sample emit) once into a graph and replay it per sweep; the proposal index and
    // the sweep come from a device counter that the graph's last node advances, so every replay is the same graph.
    // (The FP32 copy's steps are long, so with odd sweep sizes, mostly flips on small lattices, capturing costs more than
    // it saves: 1,000 chains, two sweeps of 9, 49, 81 and 225 flips take 0.84, 6.06, 13.3 and 72.4 ms with a graph and
    // 0.77, 5.84, 12.9 and 70.8 ms without.)
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    NQS_HIP_TRY(hipStreamIsCapturing(stream, &cap));
    const int n_sw = cfg.n_burnin + cfg.n_sweeps;
    if (n_sw >= 2 && (sw % 2 == 0 || cfg.dtype != NQS_F32) && cap == hipStreamCaptureStatusNone) {
        a.kbase = kbase;
        hipLaunchKernelGGL(deep_set_i64_kernel, dim3(1), dim3(1), 0, stream, kbase, (int64_t)0, (int64_t)0);
        std::string sig;
        auto add = [&](const void *p, size_t n) { sig.append((const char *)p, n); };
        add(&a, sizeof(a));
        add(&b, sizeof(b));
        add(&f, sizeof(f));
        const int64_t ints[6] = {cfg.dtype, C, sw, cfg.n_burnin, cfg.n_sweeps, N};
        add(ints, sizeof(ints));
        add(&samples, sizeof(samples));
        add(&logpsi, sizeof(logpsi));
        if (!m->sweep_exec || m->sweep_sig != sig) {
            if (m->sweep_exec) {
                // the previous graph may still run on another stream
                if (m->sweep_done) NQS_HIP_TRY(hipEventSynchronize(m->sweep_done));
                NQS_HIP_TRY(hipGraphExecDestroy(m->sweep_exec));
                m->sweep_exec = nullptr;
            }
            hipStream_t cs = capture_stream();
            if (!cs) return set_error(NQS_EDEVICE, "could not create the capture stream");
            NQS_HIP_TRY(hipStreamBeginCapture(cs, hipStreamCaptureModeRelaxed));
            for (int j = 0; j < sw; ++j) step(j, j == 0, cs);
            decide(sw, 1, 0, cs);
            if (samples || logpsi) {
                const int eb = (int)std::min<int64_t>((C * N + 255) / 256, 8192);
                hipLaunchKernelGGL(deep_emit_sweep_kernel, dim3(eb), dim3(256), 0, cs, chain_state, C, N, fcur, samples,
                                   logpsi, (const int64_t *)kbase, sw, cfg.n_burnin, cfg.n_sweeps);
            }
            hipLaunchKernelGGL(deep_set_i64_kernel, dim3(1), dim3(1), 0, cs, kbase, (int64_t)0, (int64_t)sw);
            hipGraph_t graph = nullptr;
            const hipError_t e1 = hipStreamEndCapture(cs, &graph);
            if (e1 != hipSuccess || !graph) return set_error(NQS_EDEVICE, "stream capture of the sweep failed");
            const hipError_t e2 = hipGraphInstantiate(&m->sweep_exec, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            if (e2 != hipSuccess) {
                m->sweep_exec = nullptr;
                return set_error(NQS_EDEVICE, "graph instantiation failed");
            }
            m->sweep_sig = sig;
            if (!m->sweep_done) NQS_HIP_TRY(hipEventCreateWithFlags(&m->sweep_done, hipEventDisableTiming));
        }
        for (int q = 0; q < n_sw; ++q) NQS_HIP_TRY(hipGraphLaunch(m->sweep_exec, stream));
        NQS_HIP_TRY(hipEventRecord(m->sweep_done, stream));
        if (n_accepted) hipLaunchKernelGGL(deep_copy_acc_kernel, dim3(cb), dim3(256), 0, stream, acc, C, n_accepted);
        NQS_HIP_TRY(hipGetLastError());
        return NQS_OK;
    }

    int in_sweep = 0;
    int64_t sweep = 0;
    for (int64_t k = 0; k < a.total; ++k) {
        step(k, in_sweep == 0, stream);
        if (++in_sweep == sw) {
            in_sweep = 0;
            decide(k + 1, 1, 0, stream);
            const int64_t out = sweep - cfg.n_burnin;
            if (out >= 0 && (samples || logpsi)) {
                const int eb = (int)std::min<int64_t>((C * N + 255) / 256, 8192);
                hipLaunchKernelGGL(deep_emit_kernel, dim3(eb), dim3(256), 0, stream, chain_state, C, N, fcur,
                                   samples ? samples + (size_t)out * C * N : nullptr,
                                   logpsi ? logpsi + (size_t)out * C : nullptr);
            }
            ++sweep;
        }
    }
    if (n_accepted) hipLaunchKernelGGL(deep_copy_acc_kernel, dim3(cb), dim3(256), 0, stream, acc, C, n_accepted);
    NQS_HIP_TRY(hipGetLastError());
    return NQS_OK;
}

// ---------------------------------------------------------------------------
// Local energies: rows (sample, connected configuration), a batch at a time
// ---------------------------------------------------------------------------
struct DeepElocRowsArgs {
    const int8_t *samples;
    int64_t s0;               // first sample of the batch
    int N, kind, dim, L, pbc, marshall;
    double J, h;
    int *counter;             // rows of the batch
    int *row_chain, *row_i, *row_j;
    float *row_coef;
    int *base;                // [batch] first row of each sample (its own configuration)
    int *count;               // [batch] rows of each sample
    double *diag;             // [batch]
};

// One block (256 threads) per sample of the batch.
__global__ void __launch_bounds__(256) deep_eloc_rows_kernel(DeepElocRowsArgs a)
{
    __shared__ int s_wcount[4], s_base;
    __shared__ double s_red[4];
    const int sb = blockIdx.x;
    const int64_t smp = a.s0 + sb;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int8_t *sp = a.samples + smp * a.N;
    const int nb = a.dim == 1 ? (a.pbc ? a.L : a.L - 1) : 2 * a.L * a.L;
    const int ncand = a.kind == NQS_TFIM ? a.N : 0;
    const int nloop = ncand > nb ? ncand : nb;
    // first pass: count the rows of this sample
    int mine = 0;
    double dg = 0.0;
    for (int c = tid; c < nloop; c += 256) {
        bool take = c < ncand;
        if (c < nb) {
            int bi, bj;
            bool valid = true;
            if (a.dim == 1) {
                bi = c;
                bj = c + 1 < a.L ? c + 1 : 0;
            } else {
                const int site = c >> 1, x = site / a.L, y = site % a.L;
                bi = site;
                if ((c & 1) == 0) {
                    valid = a.pbc || x + 1 < a.L;
                    bj = ((x + 1) % a.L) * a.L + y;
                } else {
                    valid = a.pbc || y + 1 < a.L;
                    bj = x * a.L + (y + 1) % a.L;
                }
            }
            if (valid) {
                dg += a.J * (double)(sp[bi] * sp[bj]);
                if (a.kind == NQS_HEISENBERG && sp[bi] != sp[bj]) take = true;
            }
        }
        mine += take ? 1 : 0;
    }
    int tot = mine;
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    if (lane == 0) s_wcount[wave] = tot;
    const double dsum = group_sum<64>(dg);
    if (lane == 0) s_red[wave] = dsum;
    __syncthreads();
    if (tid == 0) {
        const int rows = 1 + s_wcount[0] + s_wcount[1] + s_wcount[2] + s_wcount[3];
        const int b0 = atomicAdd(a.counter, rows);
        s_base = b0;
        a.base[sb] = b0;
        a.count[sb] = rows;
        a.diag[sb] = s_red[0] + s_red[1] + s_red[2] + s_red[3];
        a.row_chain[b0] = (int)smp;
        a.row_i[b0] = -1;
        a.row_j[b0] = -1;
        a.row_coef[b0] = 0.0f;
    }
    __syncthreads();
    // second pass: write the rows in candidate order
    int pos = s_base + 1;
    for (int base = 0; base < nloop; base += 256) {
        const int c = base + tid;
        int i = -1, j = -1;
        bool take = false;
        float coef = 0.0f;
        if (c < ncand) {
            i = c;
            take = true;
            coef = (float)a.h * ((a.marshall && on_sub_a(a.dim, a.L, i)) ? -1.0f : 1.0f);
        }
        if (c < nb && a.kind == NQS_HEISENBERG) {
            int bi, bj;
            bool valid = true;
            if (a.dim == 1) {
                bi = c;
                bj = c + 1 < a.L ? c + 1 : 0;
            } else {
                const int site = c >> 1, x = site / a.L, y = site % a.L;
                bi = site;
                if ((c & 1) == 0) {
                    valid = a.pbc || x + 1 < a.L;
                    bj = ((x + 1) % a.L) * a.L + y;
                } else {
                    valid = a.pbc || y + 1 < a.L;
                    bj = x * a.L + (y + 1) % a.L;
                }
            }
            if (valid && sp[bi] != sp[bj]) {
                i = bi;
                j = bj;
                take = true;
                const bool flip = a.marshall && (on_sub_a(a.dim, a.L, bi) != on_sub_a(a.dim, a.L, bj));
                coef = 2.0f * (float)a.J * (flip ? -1.0f : 1.0f);
            }
        }
        const unsigned long long bal = __ballot(take);
        __syncthreads();
        if (lane == 0) s_wcount[wave] = __popcll(bal);
        __syncthreads();
        int off = pos;
        for (int w = 0; w < wave; ++w) off += s_wcount[w];
        if (take) {
            const int r = off + __popcll(bal & ((1ull << lane) - 1ull));
            a.row_chain[r] = (int)smp;
            a.row_i[r] = i;
            a.row_j[r] = j;
            a.row_coef[r] = coef;
        }
        pos += s_wcount[0] + s_wcount[1] + s_wcount[2] + s_wcount[3];
    }
}

// One wave per sample: eps = diag + sum_rows coef exp(f_row - f_sample) (FP64).
__global__ void deep_eloc_reduce_kernel(int nb, const int *base, const int *count, const double *diag,
                                        const float *row_coef, const float *part, int npart, double *eloc)
{
    const int sb = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (sb >= nb) return;
    const int b0 = base[sb], n = count[sb];
    auto fof = [&](int r) {
        float f = 0.0f;
        for (int p = 0; p < npart; ++p) f += part[(size_t)r * npart + p];
        return f;
    };
    const float f0 = fof(b0);
    double off = 0.0;
    for (int r = 1 + lane; r < n; r += 64) off += (double)row_coef[b0 + r] * exp((double)(fof(b0 + r) - f0));
    off = group_sum<64>(off);
    if (lane == 0) eloc[sb] = diag[sb] + off;
}

nqs_status deep_local_energy(nqs_model *m, const nqs_ham_desc &ham, const int8_t *samples, int64_t n, int dtype,
                             double *eloc, hipStream_t stream)
{
    const FfnnDev &f = m->copies[dtype].ffnn;
    const int N = f.widths[0];
    const int esize = dtype == NQS_F32 ? 4 : (dtype == NQS_FP8_E4M3 ? 1 : 2);
    const int per = 2 * N + 1;                               // rows per sample at most
    const int64_t cap = std::max<int64_t>(per, std::min<int64_t>(65536, (int64_t)per * std::max<int64_t>(1, n)));
    const int bs = (int)std::max<int64_t>(1, cap / per);     // samples per batch
    const size_t fwd = deep_buffer_bytes(f, cap, esize);
    const size_t extra = al256(sizeof(float) * cap) + 2 * al256(sizeof(int) * bs) + al256(sizeof(double) * bs);
    char *ws = (char *)workspace(fwd + extra, stream);
    if (!ws) return set_error(NQS_ENOMEM, "workspace allocation failed");
    DeepBuffers b = deep_carve(f, cap, esize, ws);
    char *pe = ws + fwd;
    float *row_coef = (float *)pe;
    int *base = (int *)(pe + al256(sizeof(float) * cap));
    int *count = (int *)(pe + al256(sizeof(float) * cap) + al256(sizeof(int) * bs));
    double *diag = (double *)(pe + al256(sizeof(float) * cap) + 2 * al256(sizeof(int) * bs));

    DeepElocRowsArgs a;
    a.samples = samples;
    a.N = N;
    a.kind = ham.kind;
    a.dim = ham.dim;
    a.L = ham.L;
    a.pbc = ham.pbc;
    a.marshall = m->desc.marshall;
    a.J = ham.J;
    a.h = ham.h;
    a.counter = b.counter;
    a.row_chain = b.row_chain;
    a.row_i = b.row_i;
    a.row_j = b.row_j;
    a.row_coef = row_coef;
    a.base = base;
    a.count = count;
    a.diag = diag;
    for (int64_t s0 = 0; s0 < n; s0 += bs) {
        const int nbat = (int)std::min<int64_t>(bs, n - s0);
        a.s0 = s0;
        nqs_status z = launch_zero_u64(b.counter, 1, stream);
        if (z != NQS_OK) return z;
        hipLaunchKernelGGL(deep_eloc_rows_kernel, dim3(nbat), dim3(256), 0, stream, a);
        // a row per site (TFIM), or per unequal pair, about half of the bonds; and the sample itself
        const int64_t expect = (int64_t)nbat * (1 + (ham.kind == NQS_TFIM ? N : ham.dim * N / 2));
        deep_forward(dtype, f, b, samples, cap, expect, false, stream);
        hipLaunchKernelGGL(deep_eloc_reduce_kernel, dim3((nbat + 3) / 4), dim3(256), 0, stream, nbat, base, count, diag,
                           row_coef, b.part, b.npart, eloc + s0);
        NQS_HIP_TRY(hipGetLastError());
    }
    return NQS_OK;
}

}  // namespace nqs
