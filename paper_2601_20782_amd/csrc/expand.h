// Which factors a block of ffnn_expand_kernel (ffnn.hip) needs: the layers' weights and biases among the parameters it
// writes, and the LDS they take.  Host and device code without HIP headers.
#pragma once

#include <algorithm>
#include <cstdint>

#include "nqs.h"

namespace nqs {

struct ExpandArgs {
    const float *acts, *dels;
    float *O;                     // [n][p1 - p0]
    int64_t n, p0, p1, sa, sd;    // sa, sd: row lengths of acts and dels
    int L;
    int64_t offW[NQS_MAX_LAYERS + 1];   // first parameter of layer l; offW[L] = P
    int in[NQS_MAX_LAYERS], out[NQS_MAX_LAYERS];
    unsigned inv[NQS_MAX_LAYERS];       // of `in`, for expand_div
    int64_t offA[NQS_MAX_LAYERS], offD[NQS_MAX_LAYERS];
};

constexpr int kExpandSpan = 16384;

// q / in for a position q among a layer's weights (below 2^26), inv = (2^32 - 1) / in: the product is at most one short
__host__ __device__ inline unsigned expand_div(unsigned q, unsigned in, unsigned inv)
{
    const unsigned r = (unsigned)(((uint64_t)q * inv) >> 32);
    return q - r * in >= in ? r + 1 : r;
}

// the parameters of layer l among [b0, b1): weights [q0, q0 + count) of rows [r0, r0 + rows), biases [d0, d0 + nd)
struct ExpandPart {
    unsigned q0, count, r0;
    int rows, d0, nd;
};
__host__ __device__ inline ExpandPart expand_part(const ExpandArgs &E, int l, int64_t b0, int64_t b1)
{
    const int64_t w0 = E.offW[l], w1 = w0 + (int64_t)E.out[l] * E.in[l], w2 = E.offW[l + 1];
    const int64_t s0 = b0 > w0 ? b0 : w0, s1 = b1 < w1 ? b1 : w1, t0 = b0 > w1 ? b0 : w1, t1 = b1 < w2 ? b1 : w2;
    ExpandPart x{0u, 0u, 0u, 0, 0, 0};
    if (s0 < s1) {
        x.q0 = (unsigned)(s0 - w0);
        x.count = (unsigned)(s1 - s0);
        x.r0 = expand_div(x.q0, (unsigned)E.in[l], E.inv[l]);
        x.rows = (int)(expand_div(x.q0 + x.count - 1, (unsigned)E.in[l], E.inv[l]) - x.r0) + 1;
    }
    if (t0 < t1) {
        x.d0 = (int)(t0 - w1);
        x.nd = (int)(t1 - t0);
    }
    return x;
}

// LDS floats of a layer: its inputs if any of its weights is met, the deltas of the rows met, the biases met, each a
// multiple of 16 bytes
__host__ __device__ inline int expand_words(int in, int rows, int nd)
{
    return (rows > 0 ? ((in + 3) & ~3) + ((rows + 3) & ~3) : 0) + ((nd + 3) & ~3);
}

// LDS floats of the span that needs most.  At most kExpandSpan (rows and biases met, and the inputs of layers that lie
// within the span) and the inputs of the two layers at its ends, 8192 each: 128 KB.
inline int expand_lds_words(const ExpandArgs &E)
{
    int words = 0;
    auto span_of = [&](int64_t p) {   // the span that parameter p is in
        const int64_t b0 = E.p0 + (p - E.p0) / kExpandSpan * kExpandSpan, b1 = std::min(E.p1, b0 + kExpandSpan);
        int sum = 0;
        for (int j = 0; j < E.L; ++j) {
            const ExpandPart x = expand_part(E, j, b0, b1);
            sum += expand_words(E.in[j], x.rows, x.nd);
        }
        words = std::max(words, sum);
    };
    for (int l = 0; l < E.L; ++l) {
        if (E.offW[l + 1] <= E.p0 || E.offW[l] >= E.p1) continue;
        // a span within the weights; the spans of the first and the last of the layer's biases, and of what follows it
        words = std::max(words, expand_words(E.in[l], std::min(E.out[l], kExpandSpan / E.in[l] + 2), 0));
        for (const int64_t p : {E.offW[l + 1] - E.out[l], E.offW[l + 1] - 1, E.offW[l + 1]})
            if (p >= E.p0 && p < E.p1) span_of(p);
    }
    span_of(E.p0);
    span_of(E.p1 - 1);
    return words;
}

}  // namespace nqs
