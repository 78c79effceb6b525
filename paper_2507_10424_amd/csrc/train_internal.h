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

__device__ __forceinline__ float softplusf(float z) { return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z))); }
__device__ __forceinline__ float sigmoidf(float z) {
    const float e = expf(-fabsf(z));
    return (z >= 0.0f ? 1.0f : e) / (1.0f + e);
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
