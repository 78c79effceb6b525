// Frame counters of the persistent decoders: how workgroups take the next frame
// of a job.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ldpc {

// Frame counters.  One counter handing out every frame number would be a
// single address that every refill of every workgroup increments atomically;
// when frames stop after a few iterations, those atomics (one per frame, all
// serialised at one address) bound the decoder.  So each job has kQueues
// counters, each in a 128-byte line of its own: counter c hands out frames
// c, c + kQueues, c + 2 kQueues, ...  A workgroup draws from one counter and
// moves to another live one when it finds its counter exhausted, so all
// frames are taken before any workgroup runs out.
constexpr int kQueues = 16;
constexpr int kQueueStride = 32; // 32-bit words between counters
// the counters, then one word (in a line of its own) with a bit for every
// counter some workgroup has found exhausted
constexpr int kQueueWords = (kQueues + 1) * kQueueStride;

// Frame number of the k-th value taken from counter c of nq.
__device__ __forceinline__ int64_t frame_of(uint32_t k, int32_t c, int32_t nq) { return (int64_t)k * nq + c; }

// Counters a batch of B frames uses: one per 1,024 frames, at most kQueues
// (a small batch needs no spreading, and every counter a workgroup finds
// exhausted costs it one atomic round trip at the end).
inline int32_t queues_for(int32_t B) {
    const int32_t q = B / 1024;
    return q < 1 ? 1 : (q > kQueues ? kQueues : q);
}

// The next live counter after c, or c when none is left.
__device__ __forceinline__ int32_t next_live(int32_t c, uint32_t dead, int32_t nq) {
    for (int d = 1; d < nq; ++d) {
        const int32_t x = (c + d) % nq;
        if (!((dead >> x) & 1u)) return x;
    }
    return c;
}

// Records that counter c is exhausted and learns which others are.  Every
// workgroup comes here at the end of a batch, to one word.  PEEK: it reads the
// word, and only those that find c's bit unset yet change it ((3,6) n = 102,
// 16,000 frames, 0.121 ms without and 0.057 with); not where a GPU holds few
// workgroups and registers are full, in the LDS-resident decoder (n = 8176,
// 1,500 frames, 0.274 ms without and 0.279 with) and the two-slot kernels
// ((3,6) n = 1176, 28,863 frames, 10 iterations: 0.475 and 0.481).
template <bool PEEK> __device__ __forceinline__ uint32_t mark_dead(uint32_t *queue, int32_t c, uint32_t dead) {
    uint32_t *word = queue + kQueues * kQueueStride;
    if constexpr (PEEK) {
        const uint32_t seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!((seen >> c) & 1u)) __hip_atomic_fetch_or(word, 1u << c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return dead | (1u << c) | seen;
    } else {
        return dead | (1u << c) | atomicOr(word, 1u << c);
    }
}

// One thread: a frame number below B from the live counters (blocking), or B
// when all are exhausted.  `hc` is the counter to try first (live unless all
// are dead); each failed attempt marks at least one more counter dead, so
// the loop ends after at most nq attempts.
template <bool PEEK>
__device__ __forceinline__ int32_t take_frame(uint32_t *queue, int32_t B, int32_t nq, int32_t &hc, uint32_t &dead) {
    const uint32_t all = (1u << nq) - 1u;
    while ((dead & all) != all) {
        if ((dead >> hc) & 1u) hc = next_live(hc, dead, nq); // some counter is live
        const int64_t f = frame_of(atomicAdd(queue + hc * kQueueStride, 1u), hc, nq);
        if (f < B) return (int32_t)f;
        dead = mark_dead<PEEK>(queue, hc, dead);
    }
    return B;
}

static __global__ void k_zero_words(uint32_t *p, int32_t count) {
    const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < count) p[k] = 0u;
}

} // namespace ldpc
