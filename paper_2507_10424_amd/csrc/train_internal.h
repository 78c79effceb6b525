// Internal declarations of the training kernels (train.hip, train_lds.hip,
// train_stream.hip).
//
// Forward.  Iteration t of a check row leaves a record of the row: the two
// smallest |x| (min0 over all edges, min1 over the others), their first
// positions loc0 and loc1, and the sign bits of x.  Iteration t of a bit
// leaves its posterior s^(t).  These are all that the reverse sweep reads, so
// the backward recomputes nothing: per frame and iteration 12 bytes per row
// and 4 per bit (10 KB for n = 1024, m = 512), instead of the messages
// (4 bytes per edge) and a second forward.
//
// Backward of iteration t:
//   bits  gs_j = scale (2c_j-1) sigmoid((2c_j-1) s_j^(t)) + sum over M_j of gx_e^(t+1)
//   rows  deta_e = gs_j - gx_e^(t+1); with v0, v1 = fma(alpha, min0 / min1, -beta):
//         S0 = sum of deta_e sign_e over e != loc0 (whose magnitude is min0),
//         g0 = deta sign of loc0 (magnitude min1);
//         dalpha += [v0 > 0] S0 min0 + [v1 > 0] g0 min1,  dbeta -= [v0 > 0] S0 + [v1 > 0] g0,
//         gx^(t) = [v0 > 0] alpha S0 sign(x) at loc0, [v1 > 0] alpha g0 sign(x) at loc1, else 0.
#pragma once

#include "ldpc_internal.h"
#include "minsum_row.h"

namespace ldpc {

constexpr int kTrainMaxClasses = 8;

// exp(-|z|) as 2^-x, x = |z| log2(e) to twice the precision: the hardware's
// 2^x of the rounded x, times one plus the exponent's remainder.  (The general
// expf and log1pf take about 150 instructions for a softplus, four times a
// posterior's share of everything else; these take 25 and a sigmoid 17.  On
// 3 million values from -110 to 110 the largest relative errors are 4.6 and
// 3.8 units of 2^-24, of the library functions 4.8 and 4.3.)  NaN stays NaN.
__device__ __forceinline__ float exp_minus_abs(float z) {
    constexpr double kLog2e = 1.4426950408889634;
    constexpr float hi = (float)kLog2e, lo = (float)(kLog2e - (double)hi);
    float a = fabsf(z);
    a = a > 104.0f ? 104.0f : a; // 2^-150 and below: 0 in binary32
    const float x = a * hi;
    const float rest = fmaf(a, lo, fmaf(a, hi, -x));
    const float e = __builtin_amdgcn_exp2f(-x);
    return fmaf(e, -0.6931471805599453f * rest, e);
}
// num / d to about one unit in the last place: the hardware's reciprocal and
// one correction of the quotient (d between 1 and 3).
__device__ __forceinline__ float divide(float num, float d) {
    const float r = __builtin_amdgcn_rcpf(d), q = num * r;
    return fmaf(fmaf(-d, q, num), r, q);
}
// log1p(e) = 2 atanh(u), u = e / (2 + e) <= 1/3, by the series to u^15 (the
// next term is 1.4e-9 of the sum).
__device__ __forceinline__ float softplusf(float z) {
    const float e = exp_minus_abs(z), u = divide(e, 2.0f + e), w = u * u;
    float p = 1.0f / 15;
    p = fmaf(p, w, 1.0f / 13);
    p = fmaf(p, w, 1.0f / 11);
    p = fmaf(p, w, 1.0f / 9);
    p = fmaf(p, w, 1.0f / 7);
    p = fmaf(p, w, 1.0f / 5);
    p = fmaf(p, w, 1.0f / 3);
    const float t = u + u;
    return fmaxf(z, 0.0f) + fmaf(t * w, p, t);
}
__device__ __forceinline__ float sigmoidf(float z) {
    const float e = exp_minus_abs(z);
    return divide(z >= 0.0f ? 1.0f : e, 1.0f + e);
}

// Sum over a wavefront in a fixed order; the result in every lane.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// A call's arguments: `count` frames from frame f0 of a batch of B.
struct TrainCall {
    const float *llr;      // B x n
    const uint8_t *target; // B x n, or null
    int32_t B, f0, count, T;
    const float *alpha, *beta; // T x ncls
    float scale;               // backward: grad_loss / (B n)
    float *post, *gllr;        // B x n, or null
};

// State in LDS, a workgroup per frame (train_lds.hip).  kept: rec and s of
// every frame of the call stay in memory for the backward.
struct TrainLds {
    uint32_t *rec; // [count][T][words][row slots]
    float *s;      // [count][T][bit slots]
    float *loss_part; // [B]
    float *gpart;     // [2][T][ncls][B]
};
bool train_lds_fits(const ldpc_graph &g);
size_t train_lds_frame_bytes(const ldpc_graph &g, int32_t T); // of rec and s
size_t train_lds_rec_words(const ldpc_graph &g, int32_t T);   // of rec, per frame
int train_lds_forward(const ldpc_graph &g, const TrainCall &c, const TrainLds &w, hipStream_t s); // rec null: keep nothing
int train_lds_backward(const ldpc_graph &g, const TrainCall &c, const TrainLds &w, hipStream_t s);

// State in device memory, tiles of 64 frames with the frames innermost
// (train_stream.hip).
struct TrainStream {
    float *r, *eta, *gs, *gr; // [tile][n | E | n | n][64]; the backward keeps gx in eta
    float *s;                 // [tile][T][n][64]
    uint32_t *rec;            // [tile][T][m][words][64]
    float *loss_part;         // [T][blocks]: block_count() per iteration of the whole batch
    float *gpart;             // [2][T][ncls][waves]
};
size_t train_stream_tile_bytes(const ldpc_graph &g, int32_t T, size_t part[6]);
int64_t train_stream_loss_parts(const ldpc_graph &g, int32_t B); // per iteration
int64_t train_stream_grad_parts(const ldpc_graph &g, int32_t B); // per iteration and class
int train_stream_forward(const ldpc_graph &g, const TrainCall &c, const TrainStream &w, hipStream_t s);
int train_stream_backward(const ldpc_graph &g, const TrainCall &c, const TrainStream &w, hipStream_t s);

} // namespace ldpc
