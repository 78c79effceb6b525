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

// softplus(z) = max(z, 0) + log1p(e) and sigmoid(z), e = exp(-|z|), no less
// exact than with the general expf, log1pf and division, which take about 150
// instructions for a softplus, four times a posterior's share of everything
// else; these take 38 and a sigmoid 29.  Largest error on 3 million values each
// of |z| <= 20 and <= 110, in units of 2^-24 of the result: softplus 1.99 and
// 1.98 (general functions 2.24 and 2.20), sigmoid 2.00 and 2.00 (3.00 and
// 3.02); of results below 2^-126, 0.75 units of 2^-149 (1.00).  The hardware's
// 2^x in place of the polynomial, without the corrections of e and d, takes as
// long and had 4.6 and 3.8, and 0 below 2^-126.  NaN stays NaN.
//
// exp(-|z|) = 2^-k e^r, |r| <= ln 2 / 2, e^r = 1 + r + r^2 P(r), P of least
// largest error (0.06 units).
__device__ __forceinline__ float exp_minus_abs(float z) {
    float a = fabsf(z);
    a = a > 104.0f ? 104.0f : a; // 2^-150 and below: 0 in binary32
    const float k = rintf(a * 1.442695022e+00f);
    const float r = fmaf(k, -1.904654212e-09f, fmaf(k, 6.931471825e-01f, -a)); // ln 2 in two parts
    float p = fmaf(1.381457900e-03f, r, 8.368725888e-03f);
    p = fmaf(p, r, 4.166838899e-02f);
    p = fmaf(p, r, 1.666652113e-01f);
    p = fmaf(p, r, 4.999999404e-01f);
    return __builtin_ldexpf(1.0f + fmaf(r * r, p, r), -(int)k);
}
// num / (c + e), 1 <= c + e <= 3, as q + rest: the hardware's reciprocal, then
// what it leaves of num, with what the rounding of c + e took from it.
__device__ __forceinline__ float divide(float num, float c, float e, float &rest) {
    const float d = c + e, inv = __builtin_amdgcn_rcpf(d), q = num * inv;
    rest = fmaf(d - c - e, q, fmaf(-d, q, num)) * inv;
    return q;
}
// log1p(e) = 2 atanh(t / 2), t = 2 e / (2 + e) <= 2/3, as t + t^3 P(t^2), P of
// least largest error (0.1 units).
__device__ __forceinline__ float softplusf(float z) {
    const float e = exp_minus_abs(z);
    float rest;
    const float t = divide(e + e, 2.0f, e, rest), w = t * t;
    float p = fmaf(5.471258773e-04f, w, 2.187627135e-03f);
    p = fmaf(p, w, 1.250673085e-02f);
    p = fmaf(p, w, 8.333302289e-02f);
    return fmaxf(z, 0.0f) + (t + fmaf(t * w, p, rest));
}
__device__ __forceinline__ float sigmoidf(float z) {
    const float e = exp_minus_abs(z);
    float rest;
    const float q = divide(z >= 0.0f ? 1.0f : e, 1.0f, e, rest);
    return q + rest;
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
    float *loss_part;         // [T][parts]: train_stream_loss_parts() of the whole batch per iteration
    float *gpart;             // [2][T][ncls][waves]
};
size_t train_stream_tile_bytes(const ldpc_graph &g, int32_t T, size_t part[6]);
int64_t train_stream_loss_parts(const ldpc_graph &g, int32_t B); // per iteration
int64_t train_stream_grad_parts(const ldpc_graph &g, int32_t B); // per iteration and class
int train_stream_forward(const ldpc_graph &g, const TrainCall &c, const TrainStream &w, hipStream_t s);
int train_stream_backward(const ldpc_graph &g, const TrainCall &c, const TrainStream &w, hipStream_t s);

} // namespace ldpc
