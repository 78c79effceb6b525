// Device helpers of the kernels that keep a frame's state in LDS with the
// grouped tables of lds_tables.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ldpc {

template <class V> __device__ __forceinline__ V lds_get(const unsigned char *lds, uint32_t off) {
    return *reinterpret_cast<const V *>(lds + off);
}
template <class V> __device__ __forceinline__ void lds_put(unsigned char *lds, uint32_t off, V v) {
    *reinterpret_cast<V *>(lds + off) = v;
}
// The k-th 16-bit index of a list of pairs.
__device__ __forceinline__ uint32_t half_of(const uint32_t *w, int k) {
    return (k & 1) ? w[k >> 1] >> 16 : w[k >> 1] & 0xffffu;
}

} // namespace ldpc
