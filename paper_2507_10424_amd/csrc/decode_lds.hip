// LDS-resident Min-Sum decoder for codes that the on-chip variants do not
// take (rows of more than 16 edges, more than 1,024 rows, ...) but whose
// state (n posteriors and E messages, 4 bytes each) fits one CU's 160 KB.
//
// One workgroup of up to 1,024 threads decodes F = 1 or 2 frames in lock step
// and takes the next frame when one stops.  Rows and bits are dealt to
// wavefronts in groups of 64 of equal (or, at the seams, padded) degree:
// sorted by degree, so that a group's degree is one scalar and its code is
// unrolled for it.  Positions of the messages follow the rows: edge k of the
// row in lane l of a group sits at p0 + 64 k + l, so the check pass reads and
// writes messages at consecutive addresses and needs no per-edge registers
// for them; the bit pass gathers them.  Neighbour indices are 16-bit pairs,
// read once into registers for the first groups of a wavefront (16 words on
// either side) and streamed from the L2 for the others.
//
// Per edge and iteration the LDS serves two gathered reads, one consecutive
// read and one consecutive write, about 17 cycles per wavefront of edges with
// one frame and 24 with two (gfx950: 7 / 7.5 cycles per gathered b32 / b64
// read, 2.5 per consecutive one, 4.3 / 6.3 per write), against about 11 VALU
// instructions per frame: the LDS bounds it, which is why two frames share a
// workgroup where they fit and enough frames wait (lds_decode).  The streaming decoder moves 12 (E + n) bytes per
// frame-iteration through the Infinity Cache instead, two launches each, and
// runs a tile of 64 frames until its last one stops.  Whole calls, streaming
// before and this kernel now: n = 8176, rows of 32, 1,500 frames, 2.78 ms and
// 0.276 ms; n = 4000, rows of 2 to 14, 777 frames, 1.57 and 0.156 ms; the
// (3,6) code of n = 4096, 333 frames, 20 iterations, 0.340 and 0.071 ms.
//
// Row arithmetic, order of the sums, tests and outputs are those of the
// on-chip kernel (onchip_kernel.h); padding edges read a posterior of
// +infinity, which is never a row's minimum and never negative.
#include <algorithm>

#include "frame_queue.h"
#include "ldpc_internal.h"
#include "lds_common.h"
#include "minsum_row.h"

namespace ldpc {
namespace {

constexpr int kMaxThreads = kLdsMaxThreads;

template <int F> struct Vec;
template <> struct Vec<1> {
    typedef float type __attribute__((ext_vector_type(1)));
};
template <> struct Vec<2> {
    typedef float type __attribute__((ext_vector_type(2)));
};

struct Shared {
    int32_t next[2]; // each slot's frame after the current one
    uint32_t red[2]; // per-slot "a row is unsatisfied", by round parity
    int32_t hc;      // thread 0: the counter it draws from,
    uint32_t dead;   // and those found exhausted
};

struct LdsJob {
    LdsTables t;
    int32_t n;
    const float *llr;
    int32_t B;
    uint8_t *bits;
    float *post;
    int32_t *iters;
    uint8_t *ok;
    const float *alpha, *beta; // T x ncls, or null
    int32_t ncls;
    uint32_t *queue; // counters of the frames past the grid's first ones (zero before the launch), or null: none left
    int32_t nq;      // counters in use
};

// The rows of one group: `held` their bits' slots in registers, or `tab`
// (non-null) where to read them; `ea` the LDS address of the lane's first
// message.  al, be: the rows' weights per slot (NMS).
template <int DC, int F, bool NMS>
__device__ __forceinline__ void check_rows(unsigned char *lds, const uint32_t *held, const uint32_t *tab, uint32_t ea,
                                           const float *al, const float *be, uint32_t *usyn) {
    typedef typename Vec<F>::type V;
    constexpr uint32_t kEnt = sizeof(V);
    // Marks that differ by degree keep the compiler from merging the bodies of
    // several degrees, whose values would then all pass through copies.
    asm volatile("; rows of %0" ::"n"(DC));
    uint32_t w[(DC + 1) / 2];
#pragma unroll
    for (int k = 0; k < (DC + 1) / 2; ++k) w[k] = tab ? tab[64 * k] : held[k];
    // Eight edges at a time (four, where two frames have long rows): their
    // reads are all in flight before the first is used, and only x stays (a
    // long row's reads all at once would spill).
    constexpr int kStep = F == 2 && DC > 8 ? 4 : 8;
    V x[DC];
    uint32_t syn[F];
#pragma unroll
    for (int q = 0; q < F; ++q) syn[q] = 0u;
#pragma unroll
    for (int k0 = 0; k0 < DC; k0 += kStep) {
        V sv[kStep], ev[kStep];
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) sv[k] = lds_get<V>(lds, kEnt * half_of(w, k0 + k));
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) ev[k] = lds_get<V>(lds, ea + 64u * kEnt * (uint32_t)(k0 + k));
#pragma unroll
        for (int k = 0; k < kStep; ++k)
            if (k0 + k < DC) {
                x[k0 + k] = sv[k] - ev[k];
#pragma unroll
                for (int q = 0; q < F; ++q) {
                    if (k % 2 == 1) syn[q] = xor3(syn[q], __float_as_uint(sv[k - 1][q]), __float_as_uint(sv[k][q]));
                    else if (k0 + k + 1 == DC) syn[q] ^= __float_as_uint(sv[k][q]);
                }
            }
        if (k0 + kStep < DC) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < F; ++q) {
        uint32_t xb[DC];
        float a[DC];
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            xb[k] = __float_as_uint(x[k][q]);
            a[k] = fabsf(x[k][q]);
        }
        usyn[q] |= syn[q];
        const uint32_t par = xor_all<DC>(xb);
        float min0, min1;
        min_pair<DC>(a, min0, min1);
        if constexpr (NMS) {
            const float v0 = fmaf(al[q], min0, -be[q]), v1 = fmaf(al[q], min1, -be[q]);
            uint32_t b0 = __float_as_uint(v0 > 0.0f ? v0 : 0.0f) ^ (par & 0x80000000u);
            uint32_t b1 = __float_as_uint(v1 > 0.0f ? v1 : 0.0f) ^ (par & 0x80000000u);
#pragma unroll
            for (int k = 0; k < DC; ++k)
                x[k][q] = __uint_as_float(((a[k] == min0) ? b1 : b0) ^ (xb[k] & 0x80000000u));
        } else {
            const uint32_t K = row_word(min0, min1, par);
#pragma unroll
            for (int k = 0; k < DC; ++k) x[k][q] = edge_message(__uint_as_float(xb[k]), min1, K);
        }
    }
#pragma unroll
    for (int k = 0; k < DC; ++k) lds_put<V>(lds, ea + 64u * kEnt * (uint32_t)k, x[k]);
    asm volatile("; end of rows of %0" ::"n"(DC));
}

template <int MAXD, int F, bool NMS>
__device__ __forceinline__ void check_group(int32_t deg, unsigned char *lds, const uint32_t *held,
                                            const uint32_t *tab, uint32_t ea, const float *al, const float *be,
                                            uint32_t *usyn) {
#define LDPC_ROWS(D)                                                                                                 \
    case D:                                                                                                          \
        if constexpr (D <= MAXD) check_rows<D, F, NMS>(lds, held, tab, ea, al, be, usyn);                            \
        break;
    switch (deg) { // one scalar branch
        LDPC_ROWS(2) LDPC_ROWS(3) LDPC_ROWS(4) LDPC_ROWS(5) LDPC_ROWS(6) LDPC_ROWS(7) LDPC_ROWS(8) LDPC_ROWS(9)
        LDPC_ROWS(10) LDPC_ROWS(11) LDPC_ROWS(12) LDPC_ROWS(13) LDPC_ROWS(14) LDPC_ROWS(15) LDPC_ROWS(16)
        LDPC_ROWS(20) LDPC_ROWS(24) LDPC_ROWS(28) LDPC_ROWS(32)
    default: break;
    }
#undef LDPC_ROWS
}

// MAXD: largest row degree (8, 16 or 32).  CPT: bits per thread at most.  ALL:
// the registers hold the neighbour tables of all groups.
template <int F, int CPT, int MAXD, bool NMS, bool ALL>
__global__ __launch_bounds__(kMaxThreads) void k_lds(const LdsJob J, int32_t L, int32_t early) {
    typedef typename Vec<F>::type V;
    constexpr uint32_t kEnt = sizeof(V);
    constexpr int kRowGroups = MAXD == 32 ? 1 : 2; // groups of a wavefront with their indices in registers
    constexpr int kRowWords = MAXD / 2;
    constexpr int kBitWords = CPT <= 4 ? 4 : CPT <= 8 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int32_t n = J.n, B = J.B;
    const float *__restrict__ llr = J.llr;
    const uint32_t *__restrict__ rowtab = J.t.rows;
    const uint32_t *__restrict__ bittab = J.t.bits;
    const uint32_t eta0 = kEnt * (uint32_t)(n + 1), zero_at = eta0 + kEnt * (uint32_t)J.t.npos;
    Shared *sh = reinterpret_cast<Shared *>(lds + zero_at + kEnt);
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const int32_t w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6;

    // ---- neighbour tables in registers ---------------------------------------
    uint32_t rw[kRowGroups][kRowWords];
    int32_t rdeg[kRowGroups], rpos[kRowGroups], rcls[kRowGroups];
#pragma unroll
    for (int i = 0; i < kRowGroups; ++i) {
        const int32_t g = w + i * nw < J.t.row_groups ? w + i * nw : 0;
        const LdsGroup G = J.t.row_group[g];
        rdeg[i] = __builtin_amdgcn_readfirstlane(G.degree);
        rpos[i] = __builtin_amdgcn_readfirstlane(G.first);
        rcls[i] = NMS ? J.t.row_class[g * 64 + lane] : 0;
#pragma unroll
        for (int k = 0; k < kRowWords; ++k) // in bounds past the group's own words: the tables are padded
            rw[i][k] = rowtab[G.table + 64 * k + lane];
    }
    uint32_t bw[CPT][kBitWords];
    int32_t bdeg[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int32_t g = w + c * nw;
        bdeg[c] = 0;
        const LdsGroup G = J.t.bit_group[g < J.t.bit_groups ? g : 0];
        bdeg[c] = __builtin_amdgcn_readfirstlane(G.degree);
#pragma unroll
        for (int k = 0; k < kBitWords; ++k) bw[c][k] = bittab[G.table + 64 * k + lane];
    }

    // ---- first frames ---------------------------------------------------------
    const int32_t dealt = (int32_t)gridDim.x * F, left = B - dealt; // frames past the first ones: from the counters
    // thread 0: the next frame of a slot
    auto draw = [&](int32_t &hc, uint32_t &dead) {
        return J.queue ? dealt + take_frame<false>(J.queue, left, J.nq, hc, dead) : B;
    };
    int32_t fr[F], tt[F], ph[F];                       // ph: (tt - 1) modulo the test period
    V rc[CPT], rnx[CPT];                               // channel LLRs: own slots, next frame's own bits
#pragma unroll
    for (int q = 0; q < F; ++q) {
        fr[q] = (int32_t)blockIdx.x * F + q;
        tt[q] = 1;
        ph[q] = 0;
    }
    if (tid == 0) {
        sh->red[0] = sh->red[1] = 0u;
        int32_t hc = J.queue ? (int32_t)(blockIdx.x % (uint32_t)J.nq) : 0;
        uint32_t dead = 0u;
#pragma unroll
        for (int q = 0; q < F; ++q) sh->next[q] = draw(hc, dead);
        sh->hc = hc;
        sh->dead = dead;
    }
    const uint16_t *__restrict__ slot_of = J.t.slot_of; // of a bit
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int32_t j = tid + c * nt;
        rc[c] = 0.0f;
        rnx[c] = 0.0f;
        if (j < n) {
            V v;
#pragma unroll
            for (int q = 0; q < F; ++q)
                v[q] = fr[q] < B ? llr[(size_t)fr[q] * n + j] + 0.0f : 0.0f; // -0 -> +0
            lds_put<V>(lds, kEnt * slot_of[j], v);
        }
    }
    if (tid == 0) {
        lds_put<V>(lds, kEnt * (uint32_t)n, V(__builtin_inff()));
        lds_put<V>(lds, zero_at, V(0.0f));
    }
    for (int32_t e = tid; e < J.t.npos; e += nt) lds_put<V>(lds, eta0 + kEnt * (uint32_t)e, V(0.0f));
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int32_t p = tid + c * nt;
        if (p < n) rc[c] = lds_get<V>(lds, kEnt * (uint32_t)p);
    }
    uint32_t pend = (1u << F) - 1u; // slots whose next frame's LLRs are to be read

    for (int32_t round = 0;; ++round) {
        bool live = false;
#pragma unroll
        for (int q = 0; q < F; ++q) {
            fr[q] = __builtin_amdgcn_readfirstlane(fr[q]);
            tt[q] = __builtin_amdgcn_readfirstlane(tt[q]);
            ph[q] = __builtin_amdgcn_readfirstlane(ph[q]);
            live |= fr[q] < B;
        }
        if (!live) break;
        // Everything derived from the index words and the thread number is
        // derived again in every round: hoisted out of the loop, the decoded
        // addresses and lane masks would take several times these registers.
        int32_t tr = tid;
        asm volatile("" : "+v"(tr));
#pragma unroll
        for (int i = 0; i < kRowGroups; ++i)
#pragma unroll
            for (int k = 0; k < kRowWords; ++k) asm volatile("" : "+v"(rw[i][k]));
#pragma unroll
        for (int c = 0; c < CPT; ++c)
#pragma unroll
            for (int k = 0; k < kBitWords; ++k) asm volatile("" : "+v"(bw[c][k]));
#pragma unroll
        for (int c = 0; c < CPT; ++c) asm volatile("" : "+s"(bdeg[c]));
        const int lr = tr & 63;
        // ---- check pass ---------------------------------------------------------
        uint32_t usyn[F];
#pragma unroll
        for (int q = 0; q < F; ++q) usyn[q] = 0u;
        float al[F], be[F];
        auto weights = [&](int32_t cls) {
#pragma unroll
            for (int q = 0; q < F; ++q) {
                int32_t t = tt[q] > L ? L : tt[q]; // past the last iteration the messages are not used
                t = t < 1 ? 1 : t;
                al[q] = J.alpha[(t - 1) * J.ncls + cls];
                be[q] = J.beta[(t - 1) * J.ncls + cls];
            }
        };
#pragma unroll
        for (int i = 0; i < kRowGroups; ++i) {
            if (w + i * nw < J.t.row_groups) {
                if constexpr (NMS) weights(rcls[i]);
                check_group<MAXD, F, NMS>(rdeg[i], lds, rw[i], nullptr, eta0 + kEnt * (uint32_t)(rpos[i] + lr), al, be,
                                          usyn);
            }
        }
        for (int32_t g = w + kRowGroups * nw; !ALL && g < J.t.row_groups; g += nw) {
            const LdsGroup G = J.t.row_group[g];
            if constexpr (NMS) weights(J.t.row_class[g * 64 + lr]);
            check_group<MAXD, F, NMS>(G.degree, lds, nullptr, rowtab + G.table + lr,
                                      eta0 + kEnt * (uint32_t)(G.first + lr), al, be, usyn);
        }
        const int p = round & 1;
        uint32_t wm = 0;
#pragma unroll
        for (int q = 0; q < F; ++q) wm |= (__ballot((int32_t)usyn[q] < 0) != 0ull ? 1u : 0u) << q;
        if (lane == 0 && wm) atomicOr(&sh->red[p], wm);
        __syncthreads();
        const uint32_t U = __builtin_amdgcn_readfirstlane(sh->red[p]);
        if (tid == 0) sh->red[p ^ 1] = 0u;
        // the LLRs of the slots' next frames, read while these are decoded
        if (pend) {
#pragma unroll
            for (int q = 0; q < F; ++q) {
                if (!((pend >> q) & 1u)) continue;
                const int32_t nx = __builtin_amdgcn_readfirstlane(sh->next[q]);
                if (nx >= B) continue;
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const int32_t j = tr + c * nt;
                    rnx[c][q] = llr[(size_t)nx * n + (j < n ? j : 0)];
                }
            }
            pend = 0u;
        }
        // ---- decisions: outputs of the slots that stop -----------------------------
        uint32_t fin = 0u;
#pragma unroll
        for (int q = 0; q < F; ++q) {
            if (fr[q] >= B) continue;
            const bool clean = ((U >> q) & 1u) == 0u && ph[q] == 0 && early != 0;
            if (!(clean || tt[q] > L)) continue;
            fin |= 1u << q;
            const size_t o = (size_t)fr[q] * n;
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int32_t j = tr + c * nt;
                if (j < n) {
                    const float v = lds_get<V>(lds, kEnt * slot_of[j])[q];
                    if (J.post) J.post[o + j] = v;
                    J.bits[o + j] = v < 0.0f ? 1 : 0;
                }
            }
            if (tid == 0) {
                J.iters[fr[q]] = clean ? tt[q] - 1 : L;
                if (J.ok) J.ok[fr[q]] = ((U >> q) & 1u) == 0u ? 1 : 0;
            }
            fr[q] = __builtin_amdgcn_readfirstlane(sh->next[q]);
        }
        fin = __builtin_amdgcn_readfirstlane(fin);
#pragma unroll
        for (int q = 0; q < F; ++q) {
            const bool refilled = (fin >> q) & 1u;
            tt[q] = refilled ? 1 : tt[q] + 1;
            ph[q] = (refilled || ph[q] + 1 == early) ? 0 : ph[q] + 1;
        }
        if (fin) {
            // every thread has read its outputs and the next frame numbers
            __syncthreads();
            bool more = false;
#pragma unroll
            for (int q = 0; q < F; ++q) more |= fr[q] < B;
            if (!more) break;
            if (tid == 0) {
                int32_t hc = sh->hc;
                uint32_t dead = sh->dead;
#pragma unroll
                for (int q = 0; q < F; ++q)
                    if ((fin >> q) & 1u) sh->next[q] = draw(hc, dead);
                sh->hc = hc;
                sh->dead = dead;
            }
        }
        // ---- bit pass ---------------------------------------------------------------
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t g = w + c * nw;
            if (g < J.t.bit_groups) {
                V acc = 0.0f;
                auto msg = [&](uint32_t h) { return lds_get<V>(lds, eta0 + kEnt * h); };
                const int32_t d = bdeg[c];
                if (kBitWords >= 2 && d == 3) {
                    const V a = msg(half_of(bw[c], 0)), b = msg(half_of(bw[c], 1)), e = msg(half_of(bw[c], 2));
                    acc = a + b + e;
                } else if (d == 2) {
                    const V a = msg(half_of(bw[c], 0)), b = msg(half_of(bw[c], 1));
                    acc = a + b;
                } else if (d > 0) {
                    // pairs of messages; a group's odd last one is paired with the zero position
                    V pa[kBitWords], pb[kBitWords];
#pragma unroll
                    for (int k = 0; k < kBitWords; ++k)
                        if (2 * k < d) {
                            pa[k] = msg(half_of(&bw[c][k], 0));
                            pb[k] = msg(half_of(&bw[c][k], 1));
                        }
                    acc = pa[0] + pb[0];
#pragma unroll
                    for (int k = 1; k < kBitWords; ++k)
                        if (2 * k < d) acc = acc + pa[k] + pb[k];
                    if (!ALL && d > 2 * kBitWords) {
                        const uint32_t *tab = bittab + J.t.bit_group[g].table + lr;
                        for (int32_t k = kBitWords; 2 * k < d; ++k) {
                            const uint32_t h = tab[64 * k];
                            const V a = msg(h & 0xffffu), b = msg(h >> 16);
                            acc = acc + a + b;
                        }
                    }
                }
                const int32_t s = g * 64 + lr;
                if (s < n) lds_put<V>(lds, kEnt * (uint32_t)s, acc + rc[c]);
            }
        }
        if (fin) { // the new frames start from s = r and messages of 0
            __syncthreads();
#pragma unroll
            for (int q = 0; q < F; ++q) {
                if (!((fin >> q) & 1u)) continue;
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const int32_t j = tr + c * nt;
                    if (j < n) lds_put<float>(lds, kEnt * slot_of[j] + 4u * (uint32_t)q, fr[q] < B ? rnx[c][q] + 0.0f : 0.0f);
                }
                for (int32_t e = tr; e < J.t.npos; e += nt) lds_put<float>(lds, eta0 + kEnt * (uint32_t)e + 4u * (uint32_t)q, 0.0f);
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int32_t s = tr + c * nt;
                if (s < n) {
#pragma unroll
                    for (int q = 0; q < F; ++q)
                        if ((fin >> q) & 1u) rc[c][q] = lds_get<float>(lds, kEnt * (uint32_t)s + 4u * (uint32_t)q);
                }
            }
            pend = fin;
        }
        __syncthreads();
    }
}

using LdsFn = void (*)(const LdsJob, int32_t, int32_t);

// Bits per thread: 4, 8 or 16, the fewest that 1,024 threads need; 0 if more.
int cpt_for(const ldpc_graph &g) { return g.n <= 4 * kMaxThreads ? 4 : g.n <= 8 * kMaxThreads ? 8 : g.n <= 16 * kMaxThreads ? 16 : 0; }

size_t lds_bytes(const ldpc_graph &g, int F) {
    return 4 * (size_t)F * ((size_t)g.n + 1 + (size_t)g.lds.npos + 1) + sizeof(Shared);
}

// The kernel for F frames: rows of at most 8, 16 or 32 edges, 4, 8 or 16 bits
// per thread.  Two frames only with rows of at most 16 (a row of 32 would
// take 128 registers for its posteriors and messages alone) and at most 8
// bits per thread (more do not fit two frames in the LDS anyway).
template <bool ALL> LdsFn kernel_for(int F, int cpt, int maxd, bool nms) {
#define LDPC_K(F_, C_, D_)                                                                                           \
    if (F == F_ && cpt == C_ && maxd <= D_) return nms ? &k_lds<F_, C_, D_, true, ALL> : &k_lds<F_, C_, D_, false, ALL>;
    LDPC_K(1, 4, 8) LDPC_K(1, 4, 16) LDPC_K(1, 4, 32) LDPC_K(1, 8, 8) LDPC_K(1, 8, 16) LDPC_K(1, 8, 32)
    LDPC_K(2, 4, 8) LDPC_K(2, 8, 8)
    if constexpr (!ALL) { LDPC_K(1, 16, 32) LDPC_K(2, 4, 16) LDPC_K(2, 8, 16) }
#undef LDPC_K
    return nullptr;
}

} // namespace

bool lds_fits(const ldpc_graph &g) {
    return g.lds.rows != nullptr && cpt_for(g) != 0 && lds_bytes(g, 1) <= (size_t)g.lds_max;
}

int lds_decode(const ldpc_graph &g, const float *llr, int32_t B, int32_t L, uint32_t flags, const float *alpha,
               const float *beta, uint8_t *bits, float *post, int32_t *iters, uint8_t *ok, void *ws,
               hipStream_t stream) {
    if (!lds_fits(g)) return LDPC_EUNSUPPORTED;
    const int cpt = cpt_for(g);
    const int waves = std::min(std::max(g.lds.row_groups, (g.lds.bit_groups + cpt - 1) / cpt), kMaxThreads / 64);
    const int threads = 64 * waves;
    // What the registers hold: two groups of rows per wavefront (one of rows
    // above 16), and 8 messages of a bit (4 where a thread has 8 bits).
    const bool all = cpt <= 8 && g.lds.row_groups <= (g.dc_max > 16 ? 1 : 2) * waves && g.dv_max <= (cpt <= 4 ? 8 : 4);
    LdsFn fn = nullptr;
    size_t lds = 0;
    int64_t room = 0, promised = 0; // workgroups that the GPU holds, by the runtime's count
    auto choose = [&](int F) {
        // (two frames with rows of up to 16 spill more in the form for all groups:
        // n = 4000, 0.209 ms without it and 0.217 with it)
        fn = all && !(F == 2 && g.dc_max > 8) ? kernel_for<true>(F, cpt, g.dc_max, alpha != nullptr)
                                              : kernel_for<false>(F, cpt, g.dc_max, alpha != nullptr);
        lds = lds_bytes(g, F);
        room = resident_workgroups((const void *)fn, threads, lds, g, &promised);
        return room > 0;
    };
    if (!choose(1)) return LDPC_EHIP;
    // Two frames per workgroup where many frames wait for each: the LDS moves a
    // pair of frames for little more than one, but a frame alone finishes
    // sooner and is replaced at less cost.  Where one workgroup fills a CU and
    // rows are short, at once ((3,6) n = 4096, 1,500 frames: 0.158 ms with one
    // and 0.143 with two; (4,5) n = 1000, 10,000 frames 1.08 and 0.82); with rows
    // above 8 (whose kernel for two spills) and with four workgroups per CU and
    // more, late (irregular n = 4000: 777 frames 0.180 and 0.256 ms, 6,000 frames
    // 0.806 and 0.814; n = 1200, 256 at once and 512 by the runtime's count, 2,300
    // frames 0.224 and 0.268, 5,000 frames with two 0.417; (4,8) n = 600: 15,000 frames 0.642 and 0.766; (5,10) n =
    // 1000, 15,000 frames that do not converge: 2.17 and 1.77).  With two or three
    // per CU and short rows, only where the GPU then holds more frames, and all of
    // them or many times as many (rows of at most 8, 20 iterations: n = 1200, two
    // per CU and one of two frames, 600 frames 0.057 and 0.073 ms, 10,000 0.396
    // and 0.463; n = 1000, three and two, 800 frames 0.051 and 0.044, 1,600 0.073
    // and 0.088, 10,000 0.272 and 0.267).
    int F = 1;
    const int64_t per_cu = room / g.num_cu;
    const bool few = g.dc_max <= 8 && (per_cu == 2 || per_cu == 3);
    const int64_t alone = g.dc_max > 8 ? 8 * promised : per_cu >= 4 ? 32 * promised : room; // frames for F = 1
    if (B > alone && g.dc_max <= 16 && cpt <= 8 && lds_bytes(g, 2) <= (size_t)g.lds_max) {
        const int64_t held = room; // frames, with one per workgroup
        F = 2;
        if (!choose(2)) return LDPC_EHIP;
        if (few && (2 * room <= held || (B > 2 * room && B <= 4 * held))) {
            F = 1;
            if (!choose(1)) return LDPC_EHIP;
        }
    }
    const int64_t groups = ((int64_t)B + F - 1) / F;
    // (workgroups that wait for a CU take it as the first ones end: rows of up to
    // 16, n = 600, 800 frames 0.045 ms with 800 of which 768 run at once, 0.062 with
    // 768; n = 700, 1,100 frames 0.134 ms with 768, 0.147 with the 512 that run at once)
    const int grid = (int)std::min(groups, promised);
    LdsJob J{};
    J.t = LdsTables{g.lds.rows, g.lds.bits, g.lds.row_group, g.lds.bit_group, g.lds.slot_of, g.lds.bit_of,
                    g.lds.row_class, g.lds.row_groups, g.lds.bit_groups, g.lds.npos};
    J.n = g.n;
    J.llr = llr;
    J.B = B;
    J.bits = bits;
    J.post = post;
    J.iters = iters;
    J.ok = ok;
    J.alpha = alpha;
    J.beta = beta;
    J.ncls = (int32_t)g.class_degrees.size();
    J.queue = (int64_t)grid * F < B ? (uint32_t *)ws : nullptr; // (no smaller than the counters: any path's workspace)
    J.nq = queues_for(std::max(B, 4 * grid)); // every workgroup draws at its start
    if (J.queue) k_zero_words<<<(kQueueWords + 255) / 256, 256, 0, stream>>>(J.queue, kQueueWords);
    timed_launch(K_ONCHIP, fn, grid, threads, (uint32_t)lds, stream, J, L, test_period(flags));
    return hipGetLastError() == hipSuccess ? LDPC_OK : LDPC_EHIP;
}

} // namespace ldpc
