// Training of the learned (normalised / offset) Min-Sum decoder on the GPU.
//
// The learned decoder replaces the message magnitude mu of eq. eta_update in
// iteration t by max(fma(alpha[t-1][c], mu, -beta[t-1][c]), 0), c the degree
// class of the check row.  Training unrolls exactly T iterations (no
// syndrome exit) and minimises
//     loss = 1/(B n) sum_frames sum_{t=1..T} sum_j softplus((2 c_j - 1) s_j^(t))
// (binary cross-entropy of every iteration's posterior against the
// transmitted bits; P(bit = 1) = sigmoid(-s)).
//
// The forward runs the decoder's binary32 arithmetic (its posteriors equal
// those of ldpc_nms_decode with LDPC_NO_EARLY_EXIT bit for bit) and keeps a
// record of every row and posterior, from which the backward runs the reverse
// sweep (train_internal.h).  Frames whose state fits a workgroup's LDS are
// trained there (train_lds.hip), others in tiles of 64 with their state in
// device memory (train_stream.hip).  Sums over rows and frames are taken in a
// fixed order, so loss and gradients are the same on every run and for every
// checkpoint interval.
//
// This file: the workspace, the entry points, the sums, and the generator of
// synthetic frames and the Adam step.
//
// Measured on one MI355X (frames drawn, loss and gradients of a batch; before:
// a workgroup of 256 threads per frame, its state in LDS or in device memory,
// that kept the messages of every ckpt_every-th iteration and ran the forward
// again in between): n = 1024, 4,096 frames, T = 10: 1.97 -> 0.355 ms; n =
// 64800, 96 frames, T = 10: 51.1 -> 1.62 ms.
#include <algorithm>

#include "train_internal.h"

namespace ldpc {
namespace {

constexpr int kThreads = 256;

// Fixed-order block sum of one float per thread (wave shuffles, then the
// wave partials in order); result valid in thread 0.
__device__ float block_sum(float v, float *red) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) red[w] = v;
    __syncthreads();
    float t = 0.0f;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += red[k];
    return t;
}

// Workgroup (slice, k): the sum of slice `blockIdx.x` of gridDim.x of part[k * stride ..], times mult, to
// out0[k * gridDim.x + slice], or out1 past the first `half` outputs.  Thread i adds entries i, i + 256, ... in
// order and the block reduction adds the threads' partials in a fixed tree: the same result on every run.
__global__ __launch_bounds__(kThreads) void k_sum(const float *__restrict__ part, int64_t count, int64_t stride,
                                                  float mult, float *__restrict__ out0, float *__restrict__ out1,
                                                  int32_t half) {
    __shared__ float red[kThreads / 64];
    const int64_t slices = gridDim.x, per = (count + slices - 1) / slices, lo = per * blockIdx.x;
    const int64_t hi = lo + per < count ? lo + per : count;
    const int32_t k = blockIdx.y;
    const float *p = part + (int64_t)k * stride;
    float acc = 0.0f;
    for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) acc += p[i];
    const float tot = block_sum(acc, red);
    if (threadIdx.x == 0) {
        const int64_t o = (int64_t)k * slices + blockIdx.x;
        if (o < half) out0[o] = tot * mult;
        else out1[o - half] = tot * mult;
    }
}

// out[k] = mult * sum over i < count of part[k * stride + i] for k < width, the
// first `half` outputs to out0, the others to out1.  One workgroup per output
// up to 8,192 entries (32 per thread); more in kSumSlices slices first (tmp:
// width * kSumSlices floats), so that a long sum does not run on one CU.
constexpr int kSumSlices = 32;
void sums(const float *part, int64_t count, int64_t stride, int32_t width, float mult, float *tmp, float *out0,
          float *out1, int32_t half, hipStream_t s) {
    if (count <= 8192) {
        k_sum<<<dim3(1, width), kThreads, 0, s>>>(part, count, stride, mult, out0, out1, half);
        return;
    }
    k_sum<<<dim3(kSumSlices, width), kThreads, 0, s>>>(part, count, stride, 1.0f, tmp, tmp, INT32_MAX);
    k_sum<<<dim3(1, width), kThreads, 0, s>>>(tmp, kSumSlices, kSumSlices, mult, out0, out1, half);
}

// ---- synthetic frames --------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy
// as 1, 2, 3", SC 2011): 10 rounds of two 32x32 -> 64-bit products on a
// 128-bit counter with a 64-bit key bumped by the Weyl constants.
struct U4 {
    uint32_t x, y, z, w;
};
__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        const uint32_t lo0 = M0 * c.x, hi0 = __umulhi(M0, c.x);
        const uint32_t lo1 = M1 * c.z, hi1 = __umulhi(M1, c.z);
        c = U4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
        k0 += W0;
        k1 += W1;
    }
    return c;
}
// uniform in (0, 1]
__device__ __forceinline__ float u01(uint32_t v) { return ((float)(v >> 8) + 1.0f) * (1.0f / 16777216.0f); }

// LLRs of BPSK over AWGN for codewords (bits, or all-zero when null), with
// Eb/N0 per frame uniform in [lo_db, hi_db] (lo == hi: fixed), Box-Muller
// normals from the Philox stream keyed by `seed`; LLR = 2 y / sigma^2.
__global__ void k_awgn(const uint8_t *__restrict__ cw, int32_t B, int32_t n, float rate, float lo_db, float hi_db,
                       uint32_t seed_lo, uint32_t seed_hi, float *__restrict__ llr, float *__restrict__ ebn0_out) {
    const int32_t j0 = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    for (int32_t f = blockIdx.y; f < B; f += gridDim.y) {
        const U4 u = philox4x32_10(U4{0xFFFFFFFFu, (uint32_t)f, 0u, 0u}, seed_lo, seed_hi);
        const float eb = lo_db + (hi_db - lo_db) * (u01(u.x) - 1.0f / 16777216.0f);
        const float sigma2 = 1.0f / (2.0f * rate * exp10f(0.1f * eb));
        const float sigma = sqrtf(sigma2);
        if (ebn0_out && blockIdx.x == 0 && threadIdx.x == 0) ebn0_out[f] = eb;
        if (j0 >= n) continue;
        const U4 v = philox4x32_10(U4{(uint32_t)j0, (uint32_t)f, 1u, 0u}, seed_lo, seed_hi);
        const float r1 = sqrtf(-2.0f * logf(u01(v.x))), r2 = sqrtf(-2.0f * logf(u01(v.z)));
        const float a1 = 6.2831853071795864f * u01(v.y), a2 = 6.2831853071795864f * u01(v.w);
        const float z[4] = {r1 * cosf(a1), r1 * sinf(a1), r2 * cosf(a2), r2 * sinf(a2)};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t j = j0 + k;
            if (j < n) {
                const float x = (cw && cw[(size_t)f * n + j]) ? -1.0f : 1.0f;
                llr[(size_t)f * n + j] = 2.0f * (x + sigma * z[k]) / sigma2;
            }
        }
    }
}

// Adam (Kingma & Ba) on a flat parameter array; step is 1-based.
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m1,
                       float *__restrict__ m2, int32_t count, float lr, float b1, float b2, float eps, int32_t step) {
    const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    const float gk = g[k];
    const float a = b1 * m1[k] + (1.0f - b1) * gk;
    const float b = b2 * m2[k] + (1.0f - b2) * gk * gk;
    m1[k] = a;
    m2[k] = b;
    const float ah = a / (1.0f - powf(b1, (float)step)), bh = b / (1.0f - powf(b2, (float)step));
    p[k] -= lr * ah / (sqrtf(bh) + eps);
}

// The workspace: the forward's records and posteriors of the whole batch where
// they take no more than kKeepBytes (kSaveBytes) or than a checkpoint of the
// messages every K iterations would (with the per-frame state that such a
// backward needs); beyond that, room for the frames of one pass, and the backward
// runs the forward of each pass again.  An interval above kTimeInterval asks for
// memory rather than time (n = 1026, 8,000 frames, T = 10, intervals of 2, 3
// and 10: 902, 526 and 269 MB, 0.90, 1.19 and 1.23 ms).
constexpr size_t kKeepBytes = (size_t)8 << 30, kSaveBytes = (size_t)256 << 20;
constexpr int32_t kTimeInterval = 2;
struct Plan {
    bool lds = false;
    bool keep = true;    // the forward's records stay for the backward
    int32_t pass = 0;    // frames of a pass
    size_t unit = 0;     // bytes of a frame (lds) or a tile of 64
    size_t part[6] = {}; // of a tile's arrays
    size_t off_loss = 0, off_gpart = 0, off_tmp = 0, off_units = 0, total = 0;
    int64_t loss_parts = 0, grad_parts = 0; // streaming: per iteration (and class)
};

Plan plan_of(const ldpc_graph &g, int32_t B, int32_t T, int32_t K) {
    Plan p;
    const size_t nE = (size_t)g.n + (size_t)g.E, nck = ((size_t)T + K - 1) / K;
    const size_t ncls = g.class_degrees.size();
    p.lds = train_lds_fits(g);
    size_t budget = 4 * (size_t)B * (nck * nE + (p.lds ? 0 : 2 * nE + 2 * (size_t)g.n + K * nE));
    budget = std::max(budget, K <= kTimeInterval ? kKeepBytes : kSaveBytes);
    p.unit = p.lds ? train_lds_frame_bytes(g, T) : train_stream_tile_bytes(g, T, p.part);
    const size_t per = p.lds ? 1 : kTile, units = ((size_t)B + per - 1) / per;
    const size_t fit = std::max<size_t>(1, budget / p.unit); // frames (tiles) of a pass
    p.keep = units <= fit;
    p.pass = (int32_t)std::min<size_t>((size_t)B, fit * per);
    p.loss_parts = p.lds ? B : train_stream_loss_parts(g, B);
    p.grad_parts = p.lds ? B : train_stream_grad_parts(g, B);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    p.off_loss = take(4 * (size_t)p.loss_parts * (p.lds ? 1 : T));
    p.off_gpart = take(4 * 2 * (size_t)T * ncls * (size_t)p.grad_parts);
    p.off_tmp = take(4 * kSumSlices * std::max<size_t>(1, 2 * (size_t)T * ncls));
    // (in passes all that is allowed, so that no smaller B or T asks for more)
    p.off_units = take((p.keep ? units * p.unit : std::max(budget, p.unit)) + 6 * 256);
    p.total = off;
    return p;
}

// The arrays of `units` frames or tiles.
TrainLds lds_ws(const ldpc_graph &g, const Plan &p, int32_t T, char *base, bool records) {
    TrainLds w{};
    const size_t words = train_lds_rec_words(g, T);
    w.loss_part = (float *)(base + p.off_loss);
    w.gpart = (float *)(base + p.off_gpart);
    if (records) {
        w.rec = (uint32_t *)(base + p.off_units);
        w.s = (float *)(base + p.off_units + align_up(4 * words * (size_t)p.pass, 256));
    }
    return w;
}
TrainStream stream_ws(const Plan &p, char *base) {
    TrainStream w{};
    const size_t units = ((size_t)p.pass + kTile - 1) / kTile;
    char *b = base + p.off_units;
    auto next = [&](int k) {
        char *q = b;
        b += align_up(units * p.part[k], 256);
        return (float *)q;
    };
    w.r = next(0);
    w.eta = next(1);
    w.gs = next(2);
    w.gr = next(3);
    w.s = next(4);
    w.rec = (uint32_t *)next(5);
    w.loss_part = (float *)(base + p.off_loss);
    w.gpart = (float *)(base + p.off_gpart);
    return w;
}

// The frames of a batch in passes: fn(call of the pass).
template <class Fn> int passes(const Plan &p, TrainCall c, int32_t B, Fn fn) {
    for (int32_t f0 = 0; f0 < B; f0 += p.pass) {
        c.f0 = f0;
        c.count = std::min(p.pass, B - f0);
        const int st = fn(c);
        if (st) return st;
    }
    return LDPC_OK;
}

int train_check(const ldpc_graph *g, const float *llr, int32_t B, int32_t T, int32_t K, const float *alpha,
                const float *beta) {
    if (!g || !llr || !alpha || !beta || B < 1 || T < 1 || K < 1) return LDPC_EINVAL;
    if ((int)g->class_degrees.size() > kTrainMaxClasses) return LDPC_EUNSUPPORTED;
    return LDPC_OK;
}

} // namespace
} // namespace ldpc

using namespace ldpc;

extern "C" size_t ldpc_nms_train_workspace_bytes(const ldpc_graph *g, int32_t B, int32_t T, int32_t ckpt_every) {
    if (!g || B < 1 || T < 1 || ckpt_every < 1) return 0;
    return plan_of(*g, B, T, ckpt_every).total;
}

extern "C" int ldpc_nms_train_forward(const ldpc_graph *g, const float *llr_dev, const uint8_t *target_dev, int32_t B,
                                      int32_t T, const float *alpha_dev, const float *beta_dev, int32_t ckpt_every,
                                      float *loss_dev, float *post_dev, void *ws_dev, size_t ws_bytes,
                                      hipStream_t stream) {
    int st = train_check(g, llr_dev, B, T, ckpt_every, alpha_dev, beta_dev);
    if (st) return st;
    if (!loss_dev) return LDPC_EINVAL;
    const Plan p = plan_of(*g, B, T, ckpt_every);
    if (!ws_dev || ws_bytes < p.total) return LDPC_EWORKSPACE;
    char *base = (char *)ws_dev;
    const TrainCall call{llr_dev, target_dev, B, 0, B, T, alpha_dev, beta_dev, 0.0f, post_dev, nullptr};
    const TrainLds wl = p.lds ? lds_ws(*g, p, T, base, p.keep) : TrainLds{};
    const TrainStream wst = p.lds ? TrainStream{} : stream_ws(p, base);
    st = passes(p, call, B, [&](const TrainCall &c) {
        return p.lds ? train_lds_forward(*g, c, wl, stream) : train_stream_forward(*g, c, wst, stream);
    });
    if (st) return st;
    sums((const float *)(base + p.off_loss), p.lds ? p.loss_parts : p.loss_parts * T, 0, 1,
         1.0f / ((float)B * (float)g->n), (float *)(base + p.off_tmp), loss_dev, loss_dev, 1, stream);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

extern "C" int ldpc_nms_train_backward(const ldpc_graph *g, const float *llr_dev, const uint8_t *target_dev, int32_t B,
                                       int32_t T, const float *alpha_dev, const float *beta_dev, int32_t ckpt_every,
                                       float grad_loss, float *galpha_dev, float *gbeta_dev, float *gllr_dev,
                                       void *ws_dev, size_t ws_bytes, hipStream_t stream) {
    int st = train_check(g, llr_dev, B, T, ckpt_every, alpha_dev, beta_dev);
    if (st) return st;
    if (!galpha_dev || !gbeta_dev) return LDPC_EINVAL;
    const Plan p = plan_of(*g, B, T, ckpt_every);
    if (!ws_dev || ws_bytes < p.total) return LDPC_EWORKSPACE;
    char *base = (char *)ws_dev;
    const int32_t width = T * (int32_t)g->class_degrees.size();
    const TrainCall call{llr_dev, target_dev, B, 0, B, T, alpha_dev, beta_dev, grad_loss / ((float)B * (float)g->n),
                         nullptr, gllr_dev};
    const TrainLds wl = p.lds ? lds_ws(*g, p, T, base, true) : TrainLds{};
    const TrainStream wst = p.lds ? TrainStream{} : stream_ws(p, base);
    st = passes(p, call, B, [&](const TrainCall &c) {
        int s = LDPC_OK;
        if (!p.keep) s = p.lds ? train_lds_forward(*g, c, wl, stream) : train_stream_forward(*g, c, wst, stream);
        if (s) return s;
        return p.lds ? train_lds_backward(*g, c, wl, stream) : train_stream_backward(*g, c, wst, stream);
    });
    if (st) return st;
    sums((const float *)(base + p.off_gpart), p.grad_parts, p.grad_parts, 2 * width, 1.0f,
         (float *)(base + p.off_tmp), galpha_dev, gbeta_dev, width, stream);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

extern "C" int ldpc_awgn_llr(const uint8_t *cw_dev, int32_t B, int32_t n, float rate, float ebn0_lo_db,
                             float ebn0_hi_db, uint64_t seed, float *llr_dev, float *ebn0_dev, hipStream_t stream) {
    if (B < 0 || n < 1 || !(rate > 0.0f) || !(ebn0_hi_db >= ebn0_lo_db) || (B > 0 && !llr_dev)) return LDPC_EINVAL;
    if (B == 0) return LDPC_OK;
    const dim3 grid((unsigned)((n + 4 * 256 - 1) / (4 * 256)), (unsigned)(B < 65535 ? B : 65535));
    k_awgn<<<grid, 256, 0, stream>>>(cw_dev, B, n, rate, ebn0_lo_db, ebn0_hi_db, (uint32_t)seed,
                                     (uint32_t)(seed >> 32), llr_dev, ebn0_dev);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

extern "C" int ldpc_adam_step(float *param_dev, const float *grad_dev, float *m1_dev, float *m2_dev, int32_t count,
                              float lr, float beta1, float beta2, float eps, int32_t step, hipStream_t stream) {
    if (!param_dev || !grad_dev || !m1_dev || !m2_dev || count < 0 || step < 1) return LDPC_EINVAL;
    if (count == 0) return LDPC_OK;
    k_adam<<<(count + 255) / 256, 256, 0, stream>>>(param_dev, grad_dev, m1_dev, m2_dev, count, lr, beta1, beta2, eps,
                                                    step);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}
