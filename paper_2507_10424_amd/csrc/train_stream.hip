// Training of the learned decoder with the state in device memory, for codes
// whose frames do not fit a workgroup's LDS: tiles of 64 frames, one wavefront
// per tile and row (or bits), lane = frame, every array tile-major with the 64
// frames innermost, as in the streaming decoder (decode_stream.hip).  Each
// iteration is a row launch and a bit launch; the records and posteriors of
// every iteration (train_internal.h) stay in the workspace, so the backward is
// one bit launch and one row launch per iteration.
//
// Bound: memory.  Per frame and iteration the forward moves 12 E + 8 n bytes of
// messages and posteriors and 24 m of records (the previous messages come from
// the previous record), the backward 16 E + 8 n and 12 m.  Lanes past the batch
// load and store nothing (a last tile of 32 frames or fewer moves half the
// lines), every load of a wavefront of the bit kernels is in flight before its
// first add, and rows of at most 8 have a backward kernel of 50 registers (84
// with the rows of 16): (3,6), n = 64,800, 96 frames, per launch and iteration,
// before and after: bits 45 and 30 us, rows backward 61 and 49, rows forward
// 53 and 48, 4.2 to 5.4 TB/s.  (Two rows per wavefront, 47 us, and a tile at a
// time, whole step 1.638 ms against 1.634, gave nothing.)
#include <algorithm>

#include "train_internal.h"

namespace ldpc {
namespace {

constexpr int kWaves = 4;        // wavefronts per workgroup
constexpr int kRowsPerWave = 4;  // backward: rows whose sums one wavefront adds up
constexpr int kColsPerWave = 4;
constexpr int kMaxUnrolled = 16; // longest row that is unrolled

// Record words of a row: min0, min1, then signs | loc0 << 16 | loc1 << 24 (rows
// of at most 16 edges), else loc0, loc1 and the signs, 32 to a word.
inline int words_of(const ldpc_graph &g) { return g.dc_max <= kMaxUnrolled ? 3 : 4 + (g.dc_max + 31) / 32; }

struct Rows { // the graph in the streaming row order, where it has one
    const int32_t *row_ptr, *col_idx, *row_class;
    int32_t m, n, words;
    int64_t E;
};

// llr (B x n, frames f0 ..) -> r[tile][j][64]
__global__ __launch_bounds__(256) void k_tiles(const float *__restrict__ llr, int32_t f0, int32_t B, int32_t n,
                                               float *__restrict__ r) {
    __shared__ float t[kTile][kTile + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int32_t nchunks = (n + 63) / 64, tile = blockIdx.x / nchunks, j0 = (blockIdx.x % nchunks) * 64;
#pragma unroll 4
    for (int k = w; k < kTile; k += kWaves) {
        const int64_t f = (int64_t)f0 + tile * kTile + k;
        const int32_t j = j0 + lane;
        t[k][lane] = (f < B && j < n) ? llr[f * n + j] + 0.0f : 0.0f; // -0 -> +0
    }
    __syncthreads();
    float *rt = r + (size_t)tile * n * kTile;
#pragma unroll 4
    for (int k = w; k < kTile; k += kWaves)
        if (j0 + k < n) rt[(size_t)(j0 + k) * kTile + lane] = t[lane][k];
}

// src[tile][j][64] (tiles `stride` floats apart) -> out (B x n, frames f0 ..)
__global__ __launch_bounds__(256) void k_untile(const float *__restrict__ src, int64_t stride, int32_t f0, int32_t B,
                                                int32_t n, float *__restrict__ out) {
    __shared__ float t[kTile][kTile + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int32_t nchunks = (n + 63) / 64, tile = blockIdx.x / nchunks, j0 = (blockIdx.x % nchunks) * 64;
    const float *s = src + (size_t)tile * stride;
#pragma unroll 4
    for (int k = w; k < kTile; k += kWaves) t[lane][k] = j0 + k < n ? s[(size_t)(j0 + k) * kTile + lane] : 0.0f;
    __syncthreads();
#pragma unroll 4
    for (int k = w; k < kTile; k += kWaves) {
        const int64_t f = (int64_t)f0 + tile * kTile + k;
        if (f < B && j0 + lane < n) out[f * n + j0 + lane] = t[k][lane];
    }
}

struct Rec3 {
    float min0, min1;
    uint32_t signs, loc0, loc1;
};
__device__ __forceinline__ Rec3 rec_of(uint32_t w0, uint32_t w1, uint32_t w2) {
    return Rec3{__uint_as_float(w0), __uint_as_float(w1), w2 & 0xffffu, (w2 >> 16) & 0xffu, w2 >> 24};
}
// Weighted magnitudes of a row: the message's at every edge but loc0, and at loc0.
__device__ __forceinline__ void weigh(float al, float be, float min0, float min1, uint32_t par, uint32_t &b0,
                                      uint32_t &b1) {
    const float v0 = fmaf(al, min0, -be), v1 = fmaf(al, min1, -be);
    b0 = __float_as_uint(v0 > 0.0f ? v0 : 0.0f) ^ (par << 31);
    b1 = __float_as_uint(v1 > 0.0f ? v1 : 0.0f) ^ (par << 31);
}

// Forward check update of one row of DC edges.  al, be: this iteration's
// weights; alp, bep: the previous one's, from whose record `prev` (null in
// iteration 1) the previous messages come.
template <int DC>
__device__ __forceinline__ void row_fwd(const int32_t *__restrict__ ci, const float *__restrict__ sv,
                                        float *__restrict__ et, const uint32_t *__restrict__ prev,
                                        uint32_t *__restrict__ rec, float al, float be, float alp, float bep) {
    float s[DC], x[DC], a[DC];
#pragma unroll
    for (int k = 0; k < DC; ++k) s[k] = sv[(size_t)ci[k] * kTile];
    if (prev) {
        const Rec3 P = rec_of(prev[0], prev[kTile], prev[2 * kTile]);
        uint32_t b0, b1;
        weigh(alp, bep, P.min0, P.min1, (uint32_t)__popc(P.signs) & 1u, b0, b1);
#pragma unroll
        for (int k = 0; k < DC; ++k)
            x[k] = s[k] - __uint_as_float((P.loc0 == (uint32_t)k ? b1 : b0) ^ ((P.signs >> k) << 31));
    } else {
#pragma unroll
        for (int k = 0; k < DC; ++k) x[k] = s[k];
    }
#pragma unroll
    for (int k = 0; k < DC; ++k) a[k] = fabsf(x[k]);
    float min0, min1;
    min_pair<DC>(a, min0, min1);
    uint32_t signs = 0u, loc0 = 0u, loc1 = 0u;
#pragma unroll
    for (int k = DC - 1; k >= 0; --k) { // lowest positions win
        signs = __builtin_amdgcn_alignbit(signs, __float_as_uint(x[k]), 31);
        loc0 = a[k] == min0 ? (uint32_t)k : loc0;
    }
#pragma unroll
    for (int k = DC - 1; k >= 0; --k) loc1 = (a[k] == min1 && loc0 != (uint32_t)k) ? (uint32_t)k : loc1;
    uint32_t b0, b1;
    weigh(al, be, min0, min1, (uint32_t)__popc(signs) & 1u, b0, b1);
#pragma unroll
    for (int k = 0; k < DC; ++k)
        et[(size_t)k * kTile] = __uint_as_float((loc0 == (uint32_t)k ? b1 : b0) ^ (__float_as_uint(x[k]) & 0x80000000u));
    rec[0] = __float_as_uint(min0);
    rec[kTile] = __float_as_uint(min1);
    rec[2 * kTile] = signs | loc0 << 16 | loc1 << 24;
}

// The same for a row of any degree d in a graph with rows of more than 16
// edges: two sweeps, the signs word by word.
__device__ __forceinline__ void row_fwd_long(int32_t d, const int32_t *__restrict__ ci, const float *__restrict__ sv,
                                             float *__restrict__ et, uint32_t *__restrict__ rec, bool first, float al,
                                             float be) {
    float min0 = __builtin_inff(), min1 = __builtin_inff();
    uint32_t loc0 = 0u, loc1 = 0u, par = 0u;
    for (int32_t k0 = 0; k0 < d; k0 += 32) {
        uint32_t signs = 0u;
        for (int32_t k = k0; k < d && k < k0 + 32; ++k) {
            const float s = sv[(size_t)ci[k] * kTile];
            const float x = first ? s : s - et[(size_t)k * kTile];
            et[(size_t)k * kTile] = x;
            signs |= (__float_as_uint(x) >> 31) << (k - k0);
            const float a = fabsf(x);
            if (a < min0) {
                min1 = min0;
                loc1 = loc0;
                min0 = a;
                loc0 = (uint32_t)k;
            } else if (a < min1) {
                min1 = a;
                loc1 = (uint32_t)k;
            }
        }
        par ^= (uint32_t)__popc(signs);
        rec[(size_t)(4 + k0 / 32) * kTile] = signs;
    }
    uint32_t b0, b1;
    weigh(al, be, min0, min1, par & 1u, b0, b1);
    for (int32_t k = 0; k < d; ++k) {
        const uint32_t x = __float_as_uint(et[(size_t)k * kTile]);
        et[(size_t)k * kTile] = __uint_as_float((loc0 == (uint32_t)k ? b1 : b0) ^ (x & 0x80000000u));
    }
    rec[0] = __float_as_uint(min0);
    rec[kTile] = __float_as_uint(min1);
    rec[2 * kTile] = loc0;
    rec[3 * kTile] = loc1;
}

#define LDPC_DEGREES(X)                                                                                              \
    X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

// One wavefront = one row x one tile, iteration t.
__global__ __launch_bounds__(64 * kWaves) void k_rows_fwd(const Rows G, int32_t row_blocks, int32_t f0, int32_t B,
                                                          int32_t T, int32_t t,
                                                          const float *__restrict__ r, const float *__restrict__ s,
                                                          float *__restrict__ eta, uint32_t *__restrict__ rec,
                                                          const float *__restrict__ alpha,
                                                          const float *__restrict__ beta, int32_t ncls) {
    const uint32_t bid = xcd_swizzle(blockIdx.x, gridDim.x);
    const int32_t tile = bid / row_blocks;
    const int32_t row = (bid % row_blocks) * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= G.m || (int64_t)f0 + tile * kTile + lane >= B) return; // (lanes past the batch have no frame)
    const int32_t e0 = G.row_ptr[row], d = G.row_ptr[row + 1] - e0;
    if (d == 0) return;
    const int32_t c = G.row_class[row];
    const float al = alpha[(t - 1) * ncls + c], be = beta[(t - 1) * ncls + c];
    const int32_t tp = t > 1 ? t - 2 : 0;
    const float alp = alpha[tp * ncls + c], bep = beta[tp * ncls + c];
    const float *sv = (t == 1 ? r + (size_t)tile * G.n * kTile
                              : s + ((size_t)tile * T + (t - 2)) * G.n * kTile) + lane;
    float *et = eta + ((size_t)tile * G.E + e0) * kTile + lane;
    const size_t step = (size_t)G.m * G.words * kTile;
    uint32_t *rc = rec + ((size_t)tile * T + (t - 1)) * step + (size_t)row * G.words * kTile + lane;
    const uint32_t *prev = t > 1 ? rc - step : nullptr;
    if (G.words > 3) {
        row_fwd_long(d, G.col_idx + e0, sv, et, rc, t == 1, al, be);
        return;
    }
    switch (d) {
#define LDPC_CASE(D)                                                                                                 \
    case D: row_fwd<D>(G.col_idx + e0, sv, et, prev, rc, al, be, alp, bep); break;
        LDPC_DEGREES(LDPC_CASE)
#undef LDPC_CASE
    default: break;
    }
}

// The columns of a wavefront's four bits: their bounds and the first 8 edges of
// each, by scalar loads (both tables have 8 entries of padding, so that bits
// past n have no edges).
struct Columns {
    int32_t k0[kColsPerWave], k1[kColsPerWave], idx[kColsPerWave][8];
    __device__ __forceinline__ Columns(const int32_t *__restrict__ col_ptr, const int32_t *__restrict__ csc, int32_t c0) {
        int32_t kp[kColsPerWave + 1];
#pragma unroll
        for (int c = 0; c <= kColsPerWave; ++c) kp[c] = col_ptr[c0 + c];
#pragma unroll
        for (int c = 0; c < kColsPerWave; ++c) {
            k0[c] = kp[c];
            k1[c] = kp[c + 1];
#pragma unroll
            for (int u = 0; u < 8; ++u) idx[c][u] = csc[k0[c] + u];
        }
    }
    // Requests the first 8 values of every column of `v` (loads behind uniform
    // branches, so a column of 3 issues 3).
    __device__ __forceinline__ void load(const float *__restrict__ v, float x[kColsPerWave][8]) const {
#pragma unroll
        for (int c = 0; c < kColsPerWave; ++c)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                x[c][u] = 0.0f;
                if (k0[c] + u < k1[c]) x[c][u] = v[(size_t)idx[c][u] * kTile];
            }
    }
    // acc + the sum of column c in edge order (ascending check).
    __device__ __forceinline__ float sum(int c, const int32_t *__restrict__ csc, const float *__restrict__ v,
                                         const float x[8], float acc) const {
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = k0[c] + u < k1[c] ? acc + x[u] : acc;
        for (int32_t k = k0[c] + 8; k < k1[c]; k += 8) {
            float y[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) y[u] = v[(size_t)csc[k + u < k1[c] ? k + u : k] * kTile];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = k + u < k1[c] ? acc + y[u] : acc;
        }
        return acc;
    }
};
// Keeps the adds of the loaded values behind the last load (they stand under
// the loads' own conditions, into whose branches the compiler would move them).
__device__ __forceinline__ void all_loaded(float x[kColsPerWave][8]) {
#pragma unroll
    for (int c = 0; c < kColsPerWave; ++c)
        asm volatile("" : "+v"(x[c][0]), "+v"(x[c][1]), "+v"(x[c][2]), "+v"(x[c][3]), "+v"(x[c][4]), "+v"(x[c][5]),
                     "+v"(x[c][6]), "+v"(x[c][7]));
}

// s^(t) of four bits x one tile, and the loss of a workgroup's bits and frames.
__global__ __launch_bounds__(64 * kWaves) void k_bits_fwd(const int32_t *__restrict__ col_ptr,
                                                          const int32_t *__restrict__ csc, int32_t n, int64_t E,
                                                          int32_t col_blocks, int32_t f0, int32_t B, int32_t T,
                                                          int32_t t, const float *__restrict__ r,
                                                          const float *__restrict__ eta, float *__restrict__ s,
                                                          const uint8_t *__restrict__ target,
                                                          float *__restrict__ loss_part) {
    __shared__ float red[kWaves];
    const uint32_t bid = xcd_swizzle(blockIdx.x, gridDim.x);
    const int32_t tile = bid / col_blocks;
    const int32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t c0 = ((int32_t)(bid % col_blocks) * kWaves + w) * kColsPerWave;
    const int lane = threadIdx.x & 63;
    const int64_t f = (int64_t)f0 + tile * kTile + lane;
    const float *et = eta + (size_t)tile * E * kTile + lane, *rt = r + (size_t)tile * n * kTile + lane;
    float *st = s + ((size_t)tile * T + (t - 1)) * n * kTile + lane;
    float loss = 0.0f;
    if (c0 < n && f < B) {
        const Columns C(col_ptr, csc, c0);
        float x[kColsPerWave][8], rv[kColsPerWave];
        C.load(et, x);
#pragma unroll
        for (int c = 0; c < kColsPerWave; ++c) rv[c] = rt[(size_t)min(c0 + c, n - 1) * kTile];
        all_loaded(x);
#pragma unroll
        for (int c = 0; c < kColsPerWave; ++c) {
            const int32_t j = c0 + c;
            if (j >= n) break;
            const float v = C.sum(c, csc, et, x[c], 0.0f) + rv[c];
            st[(size_t)j * kTile] = v;
            loss += softplusf(target && target[f * n + j] ? v : -v);
        }
    }
    loss = wave_sum(loss);
    if (lane == 0) red[w] = loss;
    __syncthreads();
    if (threadIdx.x == 0) {
        float sum = 0.0f;
        for (int k = 0; k < kWaves; ++k) sum += red[k];
        loss_part[bid] = sum;
    }
}

// gs of four bits x one tile before the rows of iteration t (t = 0: gs is the
// gradient of the channel LLRs and takes no loss term).  last: no gx yet.
__global__ __launch_bounds__(64 * kWaves) void k_bits_bwd(const int32_t *__restrict__ col_ptr,
                                                          const int32_t *__restrict__ csc, int32_t n, int64_t E,
                                                          int32_t col_blocks, int32_t f0, int32_t B, int32_t T,
                                                          int32_t t, const float *__restrict__ gx,
                                                          const float *__restrict__ s,
                                                          const uint8_t *__restrict__ target, float scale,
                                                          float *__restrict__ gs, float *__restrict__ gr) {
    const uint32_t bid = xcd_swizzle(blockIdx.x, gridDim.x);
    const int32_t tile = bid / col_blocks;
    const int32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t c0 = ((int32_t)(bid % col_blocks) * kWaves + w) * kColsPerWave;
    const int lane = threadIdx.x & 63;
    const int64_t f = (int64_t)f0 + tile * kTile + lane;
    const float *gt = gx + (size_t)tile * E * kTile + lane;
    const size_t bit0 = (size_t)tile * n * kTile + lane;
    const float *st = s + ((size_t)tile * T + (t > 0 ? t - 1 : 0)) * n * kTile + lane;
    if (c0 >= n || f >= B) return;
    const Columns C(col_ptr, csc, c0);
    float x[kColsPerWave][8], sv[kColsPerWave];
    if (t < T) {
        C.load(gt, x);
    } else {
#pragma unroll
        for (int c = 0; c < kColsPerWave; ++c)
#pragma unroll
            for (int u = 0; u < 8; ++u) x[c][u] = 0.0f;
    }
#pragma unroll
    for (int c = 0; c < kColsPerWave; ++c) sv[c] = st[(size_t)min(c0 + c, n - 1) * kTile];
    all_loaded(x);
#pragma unroll
    for (int c = 0; c < kColsPerWave; ++c) {
        const int32_t j = c0 + c;
        if (j >= n) break;
        const size_t o = bit0 + (size_t)j * kTile;
        float g = 0.0f;
        if (t > 0) {
            const float y = target && target[f * n + j] ? 1.0f : -1.0f;
            g = scale * y * sigmoidf(y * sv[c]);
        } else {
            g = gr[o];
        }
        if (t < T) g = C.sum(c, csc, gt, x[c], g);
        if (t > 0) gs[o] = g;
        if (gr) gr[o] = t == T || t == 0 ? g : gr[o] + g;
    }
}

// Reverse check update of one row of DC edges.
template <int DC>
__device__ __forceinline__ void row_bwd(const int32_t *__restrict__ ci, const float *__restrict__ gs,
                                        float *__restrict__ gx, const uint32_t *__restrict__ rec, bool last, float al,
                                        float be, float &ga, float &gb) {
    const Rec3 R = rec_of(rec[0], rec[kTile], rec[2 * kTile]);
    float g[DC], x[DC];
#pragma unroll
    for (int k = 0; k < DC; ++k) g[k] = gs[(size_t)ci[k] * kTile];
#pragma unroll
    for (int k = 0; k < DC; ++k) x[k] = last ? 0.0f : gx[(size_t)k * kTile];
    const uint32_t flip = (__popc(R.signs) & 1) ? ~R.signs : R.signs;
    float S0 = 0.0f, g0 = 0.0f;
#pragma unroll
    for (int k = 0; k < DC; ++k) {
        const float d = __uint_as_float(__float_as_uint(g[k] - x[k]) ^ ((flip << (31 - k)) & 0x80000000u));
        const bool at0 = R.loc0 == (uint32_t)k;
        S0 += at0 ? 0.0f : d;
        g0 = at0 ? d : g0;
    }
    S0 = fmaf(al, R.min0, -be) > 0.0f ? S0 : 0.0f;
    g0 = fmaf(al, R.min1, -be) > 0.0f ? g0 : 0.0f;
    ga += S0 * R.min0 + g0 * R.min1;
    gb -= S0 + g0;
    const float x0 = __uint_as_float(__float_as_uint(S0 * al) ^ ((R.signs >> R.loc0) << 31));
    const float x1 = __uint_as_float(__float_as_uint(g0 * al) ^ ((R.signs >> R.loc1) << 31));
#pragma unroll
    for (int k = 0; k < DC; ++k)
        gx[(size_t)k * kTile] = R.loc0 == (uint32_t)k ? x0 : (R.loc1 == (uint32_t)k ? x1 : 0.0f);
}
__device__ __forceinline__ void row_bwd_long(int32_t d, const int32_t *__restrict__ ci, const float *__restrict__ gs,
                                             float *__restrict__ gx, const uint32_t *__restrict__ rec, bool last,
                                             float al, float be, float &ga, float &gb) {
    const float min0 = __uint_as_float(rec[0]), min1 = __uint_as_float(rec[kTile]);
    const uint32_t loc0 = rec[2 * kTile], loc1 = rec[3 * kTile];
    uint32_t par = 0u;
    for (int32_t k0 = 0; k0 < d; k0 += 32) par ^= (uint32_t)__popc(rec[(size_t)(4 + k0 / 32) * kTile]);
    float S0 = 0.0f, g0 = 0.0f;
    uint32_t neg0 = 0u, neg1 = 0u;
    for (int32_t k0 = 0; k0 < d; k0 += 32) {
        const uint32_t signs = rec[(size_t)(4 + k0 / 32) * kTile];
        for (int32_t k = k0; k < d && k < k0 + 32; ++k) {
            const uint32_t neg = (signs >> (k - k0)) & 1u;
            const float v = gs[(size_t)ci[k] * kTile] - (last ? 0.0f : gx[(size_t)k * kTile]);
            const float dv = __uint_as_float(__float_as_uint(v) ^ ((neg ^ (par & 1u)) << 31));
            if (loc0 == (uint32_t)k) {
                g0 = dv;
                neg0 = neg;
            } else {
                S0 += dv;
                if (loc1 == (uint32_t)k) neg1 = neg;
            }
        }
    }
    S0 = fmaf(al, min0, -be) > 0.0f ? S0 : 0.0f;
    g0 = fmaf(al, min1, -be) > 0.0f ? g0 : 0.0f;
    ga += S0 * min0 + g0 * min1;
    gb -= S0 + g0;
    const float x0 = __uint_as_float(__float_as_uint(S0 * al) ^ (neg0 << 31));
    const float x1 = __uint_as_float(__float_as_uint(g0 * al) ^ (neg1 << 31));
    for (int32_t k = 0; k < d; ++k)
        gx[(size_t)k * kTile] = loc0 == (uint32_t)k ? x0 : (loc1 == (uint32_t)k ? x1 : 0.0f);
}

// kRowsPerWave rows x one tile of iteration t; the wavefront's sums for every
// class go to gpart[2][T][ncls][waves].  MAXD: longest row of the graph that is
// unrolled (its registers are every wavefront's).
template <int NC, int MAXD>
__global__ __launch_bounds__(64 * kWaves) void k_rows_bwd(const Rows G, int32_t row_blocks, int32_t f0, int32_t B,
                                                          int32_t T, int32_t t,
                                                          const float *__restrict__ gs, float *__restrict__ gx,
                                                          const uint32_t *__restrict__ rec,
                                                          const float *__restrict__ alpha,
                                                          const float *__restrict__ beta, int32_t ncls,
                                                          float *__restrict__ gpart, int64_t waves, int64_t wave0) {
    const uint32_t bid = xcd_swizzle(blockIdx.x, gridDim.x);
    const int32_t tile = bid / row_blocks;
    const int32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t row0 = ((int32_t)(bid % row_blocks) * kWaves + w) * kRowsPerWave;
    const int lane = threadIdx.x & 63;
    float ga[NC], gb[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) ga[c] = gb[c] = 0.0f;
    if ((int64_t)f0 + tile * kTile + lane < B) { // lanes past the batch keep sums of zero
        for (int32_t row = row0; row < min(row0 + kRowsPerWave, G.m); ++row) {
            const int32_t e0 = G.row_ptr[row], d = G.row_ptr[row + 1] - e0;
            if (d == 0) continue;
            const int32_t cls = G.row_class[row];
            const float al = alpha[(t - 1) * ncls + cls], be = beta[(t - 1) * ncls + cls];
            const float *gv = gs + (size_t)tile * G.n * kTile + lane;
            float *xv = gx + ((size_t)tile * G.E + e0) * kTile + lane;
            const uint32_t *rc =
                rec + (((size_t)tile * T + (t - 1)) * G.m + row) * G.words * kTile + lane;
            float a = 0.0f, b = 0.0f;
            if (G.words > 3) {
                row_bwd_long(d, G.col_idx + e0, gv, xv, rc, t == T, al, be, a, b);
            } else {
                switch (d) {
#define LDPC_CASE(D)                                                                                                 \
                case D:                                                                                              \
                    if constexpr (D <= MAXD) row_bwd<D>(G.col_idx + e0, gv, xv, rc, t == T, al, be, a, b);             \
                    break;
                    LDPC_DEGREES(LDPC_CASE)
#undef LDPC_CASE
                default: break;
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (NC == 1 || cls == c) {
                    ga[c] += a;
                    gb[c] += b;
                }
        }
    }
    float *out = gpart + (int64_t)(t - 1) * ncls * waves + wave0 + (int64_t)bid * kWaves + w;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (c >= ncls) break;
        const float a = wave_sum(ga[c]), b = wave_sum(gb[c]);
        if (lane == 0) {
            out[c * waves] = a;
            out[((int64_t)T * ncls + c) * waves] = b;
        }
    }
}

using BwdFn = void (*)(const Rows, int32_t, int32_t, int32_t, int32_t, int32_t, const float *, float *,
                       const uint32_t *, const float *, const float *, int32_t, float *, int64_t, int64_t);
// (rows of more than kMaxUnrolled are not unrolled at all)
BwdFn bwd_for(const ldpc_graph &g, int32_t ncls) {
    if (g.dc_max <= 8 || g.dc_max > kMaxUnrolled) return ncls == 1 ? &k_rows_bwd<1, 8> : &k_rows_bwd<kTrainMaxClasses, 8>;
    return ncls == 1 ? &k_rows_bwd<1, kMaxUnrolled> : &k_rows_bwd<kTrainMaxClasses, kMaxUnrolled>;
}

int64_t tiles_of(int64_t frames) { return (frames + kTile - 1) / kTile; }
int32_t row_blocks(const ldpc_graph &g, int32_t per_wave) { return (g.m + kWaves * per_wave - 1) / (kWaves * per_wave); }
int32_t col_blocks(const ldpc_graph &g) { return (g.n + kWaves * kColsPerWave - 1) / (kWaves * kColsPerWave); }
// The streaming row order renumbers edges and rows alike; all its rows have
// one degree, so the row pointers stay.
Rows rows_of(const ldpc_graph &g) {
    const bool o = g.stream_order.col_idx != nullptr;
    return Rows{g.row_ptr, o ? g.stream_order.col_idx : g.col_idx, o ? g.stream_order.row_class : g.row_class, g.m, g.n,
                words_of(g), g.E};
}
const int32_t *csc_of(const ldpc_graph &g) { return g.stream_order.csc_edge ? g.stream_order.csc_edge : g.csc_edge; }

} // namespace

int64_t train_stream_loss_parts(const ldpc_graph &g, int32_t B) { return tiles_of(B) * col_blocks(g); }
int64_t train_stream_grad_parts(const ldpc_graph &g, int32_t B) {
    return tiles_of(B) * row_blocks(g, kRowsPerWave) * kWaves;
}

size_t train_stream_tile_bytes(const ldpc_graph &g, int32_t T, size_t part[6]) {
    const size_t n = (size_t)g.n * kTile * 4, e = (size_t)g.E * kTile * 4;
    const size_t p[6] = {n, e, n, n, n * T, (size_t)g.m * words_of(g) * kTile * 4 * T}; // r eta gs gr s rec
    size_t sum = 0;
    for (int k = 0; k < 6; ++k) {
        part[k] = p[k];
        sum += p[k];
    }
    return sum;
}

int train_stream_forward(const ldpc_graph &g, const TrainCall &c, const TrainStream &w, hipStream_t st) {
    const int32_t nt = (int32_t)tiles_of(c.count), nchunks = (g.n + 63) / 64, end = c.f0 + c.count;
    const int32_t rb = row_blocks(g, 1), cb = col_blocks(g), ncls = (int32_t)g.class_degrees.size();
    const Rows G = rows_of(g);
    k_tiles<<<nt * nchunks, 256, 0, st>>>(c.llr, c.f0, end, g.n, w.r);
    const int64_t parts = train_stream_loss_parts(g, c.B), part0 = (int64_t)(c.f0 / kTile) * cb;
    for (int32_t t = 1; t <= c.T; ++t) {
        k_rows_fwd<<<nt * rb, 64 * kWaves, 0, st>>>(G, rb, c.f0, end, c.T, t, w.r, w.s, w.eta, w.rec, c.alpha, c.beta,
                                                    ncls);
        k_bits_fwd<<<nt * cb, 64 * kWaves, 0, st>>>(g.col_ptr, csc_of(g), g.n, g.E, cb, c.f0, end, c.T, t, w.r, w.eta,
                                                    w.s, c.target, w.loss_part + (t - 1) * parts + part0);
    }
    if (c.post)
        k_untile<<<nt * nchunks, 256, 0, st>>>(w.s + (size_t)(c.T - 1) * g.n * kTile, (int64_t)c.T * g.n * kTile, c.f0,
                                               end, g.n, c.post);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

int train_stream_backward(const ldpc_graph &g, const TrainCall &c, const TrainStream &w, hipStream_t st) {
    const int32_t nt = (int32_t)tiles_of(c.count), nchunks = (g.n + 63) / 64, end = c.f0 + c.count;
    const int32_t rb = row_blocks(g, kRowsPerWave), cb = col_blocks(g), ncls = (int32_t)g.class_degrees.size();
    const Rows G = rows_of(g);
    const int64_t waves = train_stream_grad_parts(g, c.B), wave0 = (int64_t)(c.f0 / kTile) * rb * kWaves;
    float *gr = c.gllr ? w.gr : nullptr;
    for (int32_t t = c.T; t >= 1; --t) {
        k_bits_bwd<<<nt * cb, 64 * kWaves, 0, st>>>(g.col_ptr, csc_of(g), g.n, g.E, cb, c.f0, end, c.T, t, w.eta, w.s,
                                                    c.target, c.scale, w.gs, gr);
        auto *fn = bwd_for(g, ncls);
        fn<<<nt * rb, 64 * kWaves, 0, st>>>(G, rb, c.f0, end, c.T, t, w.gs, w.eta, w.rec, c.alpha, c.beta, ncls,
                                            w.gpart, waves, wave0);
    }
    if (gr) {
        k_bits_bwd<<<nt * cb, 64 * kWaves, 0, st>>>(g.col_ptr, csc_of(g), g.n, g.E, cb, c.f0, end, c.T, 0, w.eta, w.s,
                                                    c.target, c.scale, w.gs, gr);
        k_untile<<<nt * nchunks, 256, 0, st>>>(gr, (int64_t)g.n * kTile, c.f0, end, g.n, c.gllr);
    }
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

} // namespace ldpc
