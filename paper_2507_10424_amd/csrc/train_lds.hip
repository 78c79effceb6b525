// Training of the learned decoder with a frame's state in LDS: one workgroup
// per frame, rows and bits in the groups of lds_tables.hip, records and
// posteriors of every iteration written to memory by the forward and read by
// the backward (train_internal.h).  Workgroups walk the frames with the
// neighbour tables in registers.
//
// Bound (n = 1024, (3,6)): VALU.  Forward: 33 instructions per row and
// iteration for the check update, about 20 for the record, 3 per bit, and the
// softplus of every posterior (38); backward: about 10 per edge and the sigmoid
// (29) per bit.  Memory: 10 KB per frame and iteration written, then read
// (2.6 and 2.1 TB/s in the two kernels, 0.159 and 0.200 ms for 4,096 frames).
#include <algorithm>

#include "lds_common.h"
#include "train_internal.h"

namespace ldpc {
namespace {

constexpr int kThreads = kLdsMaxThreads;

// Bits per thread: 4, 8 or 16, the fewest that 1,024 threads need; 0 if more.
int cpt_for(const ldpc_graph &g) {
    return g.n <= 4 * kThreads ? 4 : g.n <= 8 * kThreads ? 8 : g.n <= 16 * kThreads ? 16 : 0;
}
// Record words: min0, min1, then signs | loc0 << 16 | loc1 << 24 where the
// kernel takes rows of at most 16 edges, else loc0 | loc1 << 8 and the signs.
inline int words_of(const ldpc_graph &g) { return g.dc_max <= 16 && cpt_for(g) <= 8 ? 3 : 4; }

struct Job {
    LdsTables t;
    TrainCall c;
    int32_t n, ncls;
    uint32_t *rec;
    float *s, *loss_part, *gpart;
};

struct Rec {
    float min0, min1;
    uint32_t signs, loc0, loc1;
};
template <int W> __device__ __forceinline__ Rec unpack(const uint32_t *w) {
    Rec r;
    r.min0 = __uint_as_float(w[0]);
    r.min1 = __uint_as_float(w[1]);
    if constexpr (W == 3) {
        r.signs = w[2] & 0xffffu;
        r.loc0 = (w[2] >> 16) & 0xffu;
        r.loc1 = w[2] >> 24;
    } else {
        r.loc0 = w[2] & 0xffu;
        r.loc1 = w[2] >> 8;
        r.signs = w[3];
    }
    return r;
}

// Check update of one group's rows with the record of the iteration.  Slots
// without a row read the posterior +infinity everywhere and record zeros.
template <int DC, int W>
__device__ __forceinline__ void fwd_rows(unsigned char *lds, const uint32_t *held, const uint32_t *tab, uint32_t ea,
                                         float al, float be, uint32_t *rec, int32_t slots) {
    asm volatile("; rows of %0" ::"n"(DC)); // keeps the bodies of different degrees apart
    uint32_t w[(DC + 1) / 2];
#pragma unroll
    for (int k = 0; k < (DC + 1) / 2; ++k) w[k] = tab ? tab[64 * k] : held[k];
    constexpr int kStep = 8;
    float x[DC], a[DC];
#pragma unroll
    for (int k0 = 0; k0 < DC; k0 += kStep) {
        float sv[kStep], ev[kStep];
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) sv[k] = lds_get<float>(lds, 4u * half_of(w, k0 + k));
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) ev[k] = lds_get<float>(lds, ea + 256u * (uint32_t)(k0 + k));
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) {
                x[k0 + k] = sv[k] - ev[k];
                a[k0 + k] = fabsf(x[k0 + k]);
            }
        if (k0 + kStep < DC) __builtin_amdgcn_sched_barrier(0);
    }
    float min0, min1;
    min_pair<DC>(a, min0, min1);
    uint32_t xb[DC], signs = 0u, loc0 = 0u, loc1 = 0u;
#pragma unroll
    for (int k = 0; k < DC; ++k) xb[k] = __float_as_uint(x[k]);
    const uint32_t par = xor_all<DC>(xb) & 0x80000000u;
#pragma unroll
    for (int k = DC - 1; k >= 0; --k) { // lowest positions win
        signs = __builtin_amdgcn_alignbit(signs, xb[k], 31);
        loc0 = a[k] == min0 ? (uint32_t)k : loc0;
    }
#pragma unroll
    for (int k = DC - 1; k >= 0; --k) loc1 = (a[k] == min1 && loc0 != (uint32_t)k) ? (uint32_t)k : loc1;
    const float v0 = fmaf(al, min0, -be), v1 = fmaf(al, min1, -be);
    const uint32_t b0 = __float_as_uint(v0 > 0.0f ? v0 : 0.0f) ^ par, b1 = __float_as_uint(v1 > 0.0f ? v1 : 0.0f) ^ par;
#pragma unroll
    for (int k = 0; k < DC; ++k)
        lds_put<float>(lds, ea + 256u * (uint32_t)k,
                       __uint_as_float((loc0 == (uint32_t)k ? b1 : b0) ^ (xb[k] & 0x80000000u)));
    if (rec) {
        const bool row = min0 < __builtin_inff();
        rec[0] = row ? __float_as_uint(min0) : 0u;
        rec[slots] = row ? __float_as_uint(min1) : 0u;
        if constexpr (W == 3) {
            rec[2 * slots] = signs | loc0 << 16 | loc1 << 24;
        } else {
            rec[2 * slots] = loc0 | loc1 << 8;
            rec[3 * slots] = signs;
        }
    }
    asm volatile("; end of rows of %0" ::"n"(DC));
}

// Reverse check update: gs through `w`, gx at `ea` (iteration t + 1's in, t's out).
template <int DC>
__device__ __forceinline__ void bwd_rows(unsigned char *lds, uint32_t gs0, const uint32_t *held, const uint32_t *tab,
                                         uint32_t ea, float al, float be, const Rec &R, float &ga, float &gb) {
    asm volatile("; reverse rows of %0" ::"n"(DC));
    uint32_t w[(DC + 1) / 2];
#pragma unroll
    for (int k = 0; k < (DC + 1) / 2; ++k) w[k] = tab ? tab[64 * k] : held[k];
    const uint32_t flip = (__popc(R.signs) & 1) ? ~R.signs : R.signs; // sign of the product over the other edges
    float S0 = 0.0f, g0 = 0.0f;
    constexpr int kStep = 8;
#pragma unroll
    for (int k0 = 0; k0 < DC; k0 += kStep) {
        float gv[kStep], gx[kStep];
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) gv[k] = lds_get<float>(lds, gs0 + 4u * half_of(w, k0 + k));
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) gx[k] = lds_get<float>(lds, ea + 256u * (uint32_t)(k0 + k));
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) {
                const uint32_t kk = (uint32_t)(k0 + k);
                const float d =
                    __uint_as_float(__float_as_uint(gv[k] - gx[k]) ^ ((flip << (31u - kk)) & 0x80000000u));
                const bool at0 = R.loc0 == kk;
                S0 += at0 ? 0.0f : d;
                g0 = at0 ? d : g0;
            }
        if (k0 + kStep < DC) __builtin_amdgcn_sched_barrier(0);
    }
    S0 = fmaf(al, R.min0, -be) > 0.0f ? S0 : 0.0f;
    g0 = fmaf(al, R.min1, -be) > 0.0f ? g0 : 0.0f;
    ga += S0 * R.min0 + g0 * R.min1;
    gb -= S0 + g0;
    const float x0 = __uint_as_float(__float_as_uint(S0 * al) ^ ((R.signs >> R.loc0) << 31));
    const float x1 = __uint_as_float(__float_as_uint(g0 * al) ^ ((R.signs >> R.loc1) << 31));
#pragma unroll
    for (int k = 0; k < DC; ++k)
        lds_put<float>(lds, ea + 256u * (uint32_t)k,
                       R.loc0 == (uint32_t)k ? x0 : (R.loc1 == (uint32_t)k ? x1 : 0.0f));
    asm volatile("; end of reverse rows of %0" ::"n"(DC));
}

#define LDPC_DEGREES(X)                                                                                              \
    X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(20) X(24) X(28) X(32)

template <int MAXD, int W>
__device__ __forceinline__ void fwd_group(int32_t deg, unsigned char *lds, const uint32_t *held, const uint32_t *tab,
                                          uint32_t ea, float al, float be, uint32_t *rec, int32_t slots) {
    switch (deg) { // one scalar branch
#define LDPC_CASE(D)                                                                                                 \
    case D:                                                                                                          \
        if constexpr (D <= MAXD) fwd_rows<D, W>(lds, held, tab, ea, al, be, rec, slots);                             \
        break;
        LDPC_DEGREES(LDPC_CASE)
#undef LDPC_CASE
    default: break;
    }
}
template <int MAXD>
__device__ __forceinline__ void bwd_group(int32_t deg, unsigned char *lds, uint32_t gs0, const uint32_t *held,
                                          const uint32_t *tab, uint32_t ea, float al, float be, const Rec &R,
                                          float &ga, float &gb) {
    switch (deg) {
#define LDPC_CASE(D)                                                                                                 \
    case D:                                                                                                          \
        if constexpr (D <= MAXD) bwd_rows<D>(lds, gs0, held, tab, ea, al, be, R, ga, gb);                            \
        break;
        LDPC_DEGREES(LDPC_CASE)
#undef LDPC_CASE
    default: break;
    }
}

// The sum over a bit's message list of the values at `base`, in ascending
// check order from `acc`.  KW words of pairs are held; the rest is read.
// ALL: nothing is left to read.
template <int KW, bool ALL>
__device__ __forceinline__ float column_sum(const unsigned char *lds, uint32_t base, int32_t d, const uint32_t *held,
                                            const uint32_t *tab, float acc) {
    float a[KW], b[KW];
#pragma unroll
    for (int k = 0; k < KW; ++k)
        if (2 * k < d) { // (a group's odd last entry is paired with the zero position)
            a[k] = lds_get<float>(lds, base + 4u * (held[k] & 0xffffu));
            b[k] = lds_get<float>(lds, base + 4u * (held[k] >> 16));
        }
#pragma unroll
    for (int k = 0; k < KW; ++k)
        if (2 * k < d) acc = acc + a[k] + b[k];
    if constexpr (!ALL)
        for (int32_t k = KW; 2 * k < d; ++k) {
            const uint32_t h = tab[64 * k];
            const float u = lds_get<float>(lds, base + 4u * (h & 0xffffu));
            const float v = lds_get<float>(lds, base + 4u * (h >> 16));
            acc = acc + u + v;
        }
    return acc;
}

// Neighbour tables of a wavefront's first groups, in registers: LEAST for graphs
// with one group of rows per wavefront and bits of at most 4 messages.
template <int CPT, int MAXD, bool LEAST> struct Held {
    static constexpr int kRowGroups = MAXD == 32 || LEAST ? 1 : 2, kRowWords = MAXD / 2;
    static constexpr int kBitWords = CPT <= 4 && !LEAST ? 4 : CPT <= 8 ? 2 : 1;
    uint32_t rw[kRowGroups][kRowWords], bw[CPT][kBitWords];
    int32_t rdeg[kRowGroups], rpos[kRowGroups], rcls[kRowGroups], bdeg[CPT];
    __device__ __forceinline__ void load(const LdsTables &t, int32_t w, int32_t nw, int lane) {
#pragma unroll
        for (int i = 0; i < kRowGroups; ++i) {
            const int32_t g = w + i * nw < t.row_groups ? w + i * nw : 0;
            const LdsGroup G = t.row_group[g];
            rdeg[i] = __builtin_amdgcn_readfirstlane(G.degree);
            rpos[i] = __builtin_amdgcn_readfirstlane(G.first);
            rcls[i] = t.row_class[g * 64 + lane];
#pragma unroll
            for (int k = 0; k < kRowWords; ++k) rw[i][k] = t.rows[G.table + 64 * k + lane]; // (the tables are padded)
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t g = w + c * nw;
            const LdsGroup G = t.bit_group[g < t.bit_groups ? g : 0];
            bdeg[c] = __builtin_amdgcn_readfirstlane(G.degree);
#pragma unroll
            for (int k = 0; k < kBitWords; ++k) bw[c][k] = t.bits[G.table + 64 * k + lane];
        }
    }
    // Makes the words and the thread number opaque, so that what is derived
    // from them (addresses, lane masks) is derived again in every iteration
    // instead of kept in registers.  Returns the thread number.
    __device__ __forceinline__ int again(int tid) {
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int i = 0; i < kRowGroups; ++i)
#pragma unroll
            for (int k = 0; k < kRowWords; ++k) asm volatile("" : "+v"(rw[i][k]));
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
#pragma unroll
            for (int k = 0; k < kBitWords; ++k) asm volatile("" : "+v"(bw[c][k]));
            asm volatile("" : "+s"(bdeg[c]));
        }
        return tid;
    }
};

// What the registers hold of the neighbour tables: some groups', all groups',
// all groups' where LEAST suffices.
enum Tables { kSome, kAll, kLeast };
// Waves per SIMD asked for: the smallest form is bound by latency with the four
// that the compiler's own choice of registers leaves (a step of n = 1024, 4,096
// frames: 0.424 ms with four, 0.367 with six, 0.379 with eight); the others
// would spill too much.
constexpr int waves_for(int tables) { return tables == kLeast ? 6 : 1; }

template <int CPT, int MAXD, int TAB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(waves_for(TAB)))) void k_train_fwd(const Job J) {
    constexpr int W = MAXD <= 16 ? 3 : 4;
    constexpr bool ALL = TAB != kSome;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int32_t n = J.n, T = J.c.T, slots = 64 * J.t.row_groups, bslots = 64 * J.t.bit_groups;
    const uint32_t eta0 = 4u * (uint32_t)(n + 1), zero_at = eta0 + 4u * (uint32_t)J.t.npos;
    float *red = reinterpret_cast<float *>(lds + zero_at + 4u);
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const int32_t w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6;
    typedef Held<CPT, MAXD, TAB == kLeast> H;
    H h;
    h.load(J.t, w, nw, lane);
    uint32_t at[CPT]; // slots of the bits tid + c nt
#pragma unroll
    for (int c = 0; c < CPT; ++c) at[c] = tid + c * nt < n ? J.t.slot_of[tid + c * nt] : 0u;
    if (tid == 0) {
        lds_put<float>(lds, 4u * (uint32_t)n, __builtin_inff());
        lds_put<float>(lds, zero_at, 0.0f);
    }
    for (int32_t i = blockIdx.x; i < J.c.count; i += gridDim.x) {
        const size_t f = (size_t)J.c.f0 + i;
        const int tf = h.again(tid);
        float rc[CPT];
        uint32_t ones = 0u; // own slots whose transmitted bit is 1
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t j = tf + c * nt;
            if (j < n) lds_put<float>(lds, 4u * at[c], J.c.llr[f * n + j] + 0.0f); // -0 -> +0
        }
        for (int32_t e = tf; e < J.t.npos; e += nt) lds_put<float>(lds, eta0 + 4u * (uint32_t)e, 0.0f);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t p = tf + c * nt;
            rc[c] = p < n ? lds_get<float>(lds, 4u * (uint32_t)p) : 0.0f;
            if (J.c.target && p < n && J.c.target[f * n + J.t.bit_of[p]]) ones |= 1u << c;
        }
        uint32_t *rec = J.rec ? J.rec + (size_t)i * T * W * slots : nullptr;
        float *sv = J.rec ? J.s + (size_t)i * T * bslots : nullptr;
        float lacc = 0.0f;
        for (int32_t t = 1; t <= T; ++t) {
            const int tr = h.again(tid), lr = tr & 63;
            const float *al = J.c.alpha + (t - 1) * J.ncls, *be = J.c.beta + (t - 1) * J.ncls;
#pragma unroll
            for (int q = 0; q < H::kRowGroups; ++q) {
                const int32_t g = w + q * nw;
                if (g < J.t.row_groups)
                    fwd_group<MAXD, W>(h.rdeg[q], lds, h.rw[q], nullptr, eta0 + 4u * (uint32_t)(h.rpos[q] + lr),
                                       al[h.rcls[q]], be[h.rcls[q]], rec ? rec + 64 * g + lr : nullptr, slots);
            }
            for (int32_t g = w + H::kRowGroups * nw; !ALL && g < J.t.row_groups; g += nw) {
                const LdsGroup G = J.t.row_group[g];
                const int32_t cls = J.t.row_class[g * 64 + lr];
                fwd_group<MAXD, W>(G.degree, lds, nullptr, J.t.rows + G.table + lr,
                                   eta0 + 4u * (uint32_t)(G.first + lr), al[cls], be[cls],
                                   rec ? rec + 64 * g + lr : nullptr, slots);
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int32_t g = w + c * nw, p = tr + c * nt;
                if (g < J.t.bit_groups) {
                    const float s = column_sum<H::kBitWords, ALL>(lds, eta0, h.bdeg[c], h.bw[c],
                                                             ALL ? nullptr : J.t.bits + J.t.bit_group[g].table + lr, 0.0f) +
                                    rc[c];
                    if (p < n) {
                        lds_put<float>(lds, 4u * (uint32_t)p, s);
                        lacc += softplusf((ones >> c) & 1u ? s : -s);
                    }
                    if (sv) sv[p] = s;
                }
            }
            if (rec) {
                rec += (size_t)W * slots;
                sv += bslots;
            }
            __syncthreads();
        }
        if (J.c.post) {
            const int tp = h.again(tid);
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int32_t j = tp + c * nt;
                if (j < n) J.c.post[f * n + j] = lds_get<float>(lds, 4u * at[c]);
            }
        }
        const float ws = wave_sum(lacc);
        if (lane == 0) red[w] = ws;
        __syncthreads();
        if (tid == 0) {
            float sum = 0.0f;
            for (int32_t k = 0; k < nw; ++k) sum += red[k];
            J.loss_part[f] = sum;
        }
    }
}

// NC: degree classes, 1 or up to kTrainMaxClasses.
template <int CPT, int MAXD, int NC, int TAB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(waves_for(TAB)))) void k_train_bwd(const Job J) {
    constexpr int W = MAXD <= 16 ? 3 : 4;
    constexpr bool ALL = TAB != kSome;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int32_t n = J.n, T = J.c.T, B = J.c.B, slots = 64 * J.t.row_groups, bslots = 64 * J.t.bit_groups;
    const uint32_t gx0 = 4u * (uint32_t)(n + 1), zero_at = gx0 + 4u * (uint32_t)J.t.npos; // gs first, then gx
    float *red = reinterpret_cast<float *>(lds + zero_at + 4u);                            // [wave][2 NC]
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const int32_t w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6;
    typedef Held<CPT, MAXD, TAB == kLeast> H;
    H h;
    h.load(J.t, w, nw, lane);
    if (tid == 0) {
        lds_put<float>(lds, 4u * (uint32_t)n, 0.0f);
        lds_put<float>(lds, zero_at, 0.0f);
    }
    for (int32_t i = blockIdx.x; i < J.c.count; i += gridDim.x) {
        const size_t f = (size_t)J.c.f0 + i;
        const int tf = h.again(tid);
        float gr[CPT];
        uint32_t ones = 0u;
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t p = tf + c * nt;
            gr[c] = 0.0f;
            if (J.c.target && p < n && J.c.target[f * n + J.t.bit_of[p]]) ones |= 1u << c;
        }
        for (int32_t e = tf; e < J.t.npos; e += nt) lds_put<float>(lds, gx0 + 4u * (uint32_t)e, 0.0f);
        const uint32_t *rec = J.rec + ((size_t)i * T + T - 1) * W * slots;
        const float *sv = J.s + ((size_t)i * T + T - 1) * bslots;
        float sn[CPT]; // the posteriors of the next bit pass, read one pass ahead
#pragma unroll
        for (int c = 0; c < CPT; ++c) sn[c] = w + c * nw < J.t.bit_groups ? sv[tf + c * nt] : 0.0f;
        __syncthreads();
        for (int32_t t = T; t >= 1; --t) {
            const int tr = h.again(tid), lr = tr & 63;
            // the records of the held rows, read ahead of their pass
            uint32_t rn[H::kRowGroups][W];
#pragma unroll
            for (int q = 0; q < H::kRowGroups; ++q) {
                const int32_t g = w + q * nw < J.t.row_groups ? w + q * nw : 0;
#pragma unroll
                for (int k = 0; k < W; ++k) rn[q][k] = rec[(size_t)k * slots + 64 * g + lr];
            }
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int32_t g = w + c * nw, p = tr + c * nt;
                if (g < J.t.bit_groups) {
                    const float y = (ones >> c) & 1u ? 1.0f : -1.0f;
                    const float gj = column_sum<H::kBitWords, ALL>(lds, gx0, h.bdeg[c], h.bw[c],
                                                              ALL ? nullptr : J.t.bits + J.t.bit_group[g].table + lr,
                                                              J.c.scale * y * sigmoidf(y * sn[c]));
                    gr[c] += gj;
                    if (p < n) lds_put<float>(lds, 4u * (uint32_t)p, gj);
                }
            }
            if (t > 1) {
                sv -= bslots;
#pragma unroll
                for (int c = 0; c < CPT; ++c) sn[c] = w + c * nw < J.t.bit_groups ? sv[tr + c * nt] : 0.0f;
            }
            __syncthreads();
            float ga[NC], gb[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) ga[c] = gb[c] = 0.0f;
            const float *al = J.c.alpha + (t - 1) * J.ncls, *be = J.c.beta + (t - 1) * J.ncls;
            auto rows = [&](int32_t deg, const uint32_t *held, const uint32_t *tab, uint32_t pos, int32_t cls,
                            const uint32_t *rw) {
                float a = 0.0f, b = 0.0f;
                bwd_group<MAXD>(deg, lds, 0u, held, tab, gx0 + 4u * (pos + (uint32_t)lr), al[cls], be[cls],
                                unpack<W>(rw), a, b);
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (NC == 1 || cls == c) {
                        ga[c] += a;
                        gb[c] += b;
                    }
            };
#pragma unroll
            for (int q = 0; q < H::kRowGroups; ++q)
                if (w + q * nw < J.t.row_groups)
                    rows(h.rdeg[q], h.rw[q], nullptr, (uint32_t)h.rpos[q], h.rcls[q], rn[q]);
            for (int32_t g = w + H::kRowGroups * nw; !ALL && g < J.t.row_groups; g += nw) {
                const LdsGroup G = J.t.row_group[g];
                uint32_t rw[W];
#pragma unroll
                for (int k = 0; k < W; ++k) rw[k] = rec[(size_t)k * slots + 64 * g + lr];
                rows(G.degree, nullptr, J.t.rows + G.table + lr, (uint32_t)G.first, J.t.row_class[g * 64 + lr], rw);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const float a = wave_sum(ga[c]), b = wave_sum(gb[c]);
                if (lane == 0) {
                    red[2 * NC * w + c] = a;
                    red[2 * NC * w + NC + c] = b;
                }
            }
            rec -= (size_t)W * slots;
            __syncthreads();
            if (tid < 2 * NC) { // (the next write to red is past the next barrier)
                const int32_t c = tid % NC;
                float sum = 0.0f;
                for (int32_t k = 0; k < nw; ++k) sum += red[2 * NC * k + tid];
                if (c < J.ncls) J.gpart[((size_t)(tid / NC) * T * J.ncls + (size_t)(t - 1) * J.ncls + c) * B + f] = sum;
            }
        }
        if (J.c.gllr) { // x^(1) = r: the last gx goes to the channel LLRs too
            const int tg = h.again(tid);
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int32_t g = w + c * nw, p = tg + c * nt;
                if (g < J.t.bit_groups) {
                    const float v = column_sum<H::kBitWords, ALL>(lds, gx0, h.bdeg[c], h.bw[c],
                                                             ALL ? nullptr : J.t.bits + J.t.bit_group[g].table + (tg & 63), gr[c]);
                    if (p < n) J.c.gllr[f * n + J.t.bit_of[p]] = v;
                }
            }
        }
        __syncthreads();
    }
}

using Fn = void (*)(const Job);

// n + 1 posteriors (gs), npos + 1 messages (gx), 2 sums per wavefront and class
size_t lds_bytes(const ldpc_graph &g) {
    return 4 * ((size_t)g.n + 1 + (size_t)g.lds.npos + 1 + 2 * kTrainMaxClasses * (kThreads / 64));
}

// Rows of at most 8, 16 or 32 edges; 4, 8 or 16 bits per thread.
Fn kernel_for(bool fwd, int cpt, int maxd, int ncls, int tables) {
#define LDPC_K(C_, D_, T_)                                                                                           \
    if (cpt == C_ && maxd <= D_ && tables == T_)                                                                     \
        return fwd ? &k_train_fwd<C_, D_, T_>                                                                        \
                   : ncls == 1 ? &k_train_bwd<C_, D_, 1, T_> : &k_train_bwd<C_, D_, kTrainMaxClasses, T_>;
    LDPC_K(4, 8, kLeast)
    LDPC_K(4, 8, kAll) LDPC_K(4, 16, kAll) LDPC_K(4, 32, kAll) LDPC_K(8, 8, kAll) LDPC_K(8, 16, kAll)
    LDPC_K(8, 32, kAll)
    LDPC_K(4, 8, kSome) LDPC_K(4, 16, kSome) LDPC_K(4, 32, kSome) LDPC_K(8, 8, kSome) LDPC_K(8, 16, kSome)
    LDPC_K(8, 32, kSome) LDPC_K(16, 32, kSome)
#undef LDPC_K
    return nullptr;
}

// The registers hold two groups of rows per wavefront (one of rows above 16) and
// 8 messages of a bit (4 where a thread has 8 bits), or (kLeast) one group of
// rows of at most 8 and 4 messages.
int tables_for(const ldpc_graph &g, int cpt, int waves) {
    if (cpt == 4 && g.dc_max <= 8 && g.dv_max <= 4 && g.lds.row_groups <= waves) return kLeast;
    return cpt <= 8 && g.lds.row_groups <= (g.dc_max > 16 ? 1 : 2) * waves && g.dv_max <= (cpt <= 4 ? 8 : 4) ? kAll
                                                                                                            : kSome;
}

int launch(const ldpc_graph &g, const TrainCall &c, const TrainLds &w, bool fwd, hipStream_t s) {
    const int cpt = cpt_for(g);
    const int ncls = (int)g.class_degrees.size();
    const int waves = std::min(std::max(g.lds.row_groups, (g.lds.bit_groups + cpt - 1) / cpt), kThreads / 64);
    const int threads = 64 * waves;
    const Fn fn = kernel_for(fwd, cpt, g.dc_max, ncls, tables_for(g, cpt, waves));
    const size_t lds = lds_bytes(g);
    const int64_t room = resident_workgroups((const void *)fn, threads, lds, g);
    if (room < 0) return LDPC_EHIP;
    Job J{};
    J.t = LdsTables{g.lds.rows, g.lds.bits, g.lds.row_group, g.lds.bit_group, g.lds.slot_of, g.lds.bit_of,
                    g.lds.row_class, g.lds.row_groups, g.lds.bit_groups, g.lds.npos};
    J.c = c;
    J.n = g.n;
    J.ncls = ncls;
    J.rec = w.rec;
    J.s = w.s;
    J.loss_part = w.loss_part;
    J.gpart = w.gpart;
    fn<<<(unsigned)std::min<int64_t>(room, c.count), threads, lds, s>>>(J);
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

} // namespace

bool train_lds_fits(const ldpc_graph &g) {
    return g.lds.rows != nullptr && cpt_for(g) != 0 && lds_bytes(g) <= (size_t)g.lds_max;
}
size_t train_lds_rec_words(const ldpc_graph &g, int32_t T) {
    return (size_t)T * words_of(g) * 64 * (size_t)g.lds.row_groups;
}
size_t train_lds_frame_bytes(const ldpc_graph &g, int32_t T) {
    return 4 * (train_lds_rec_words(g, T) + (size_t)T * 64 * (size_t)g.lds.bit_groups);
}
int train_lds_forward(const ldpc_graph &g, const TrainCall &c, const TrainLds &w, hipStream_t s) {
    return launch(g, c, w, true, s);
}
int train_lds_backward(const ldpc_graph &g, const TrainCall &c, const TrainLds &w, hipStream_t s) {
    return launch(g, c, w, false, s);
}

} // namespace ldpc
