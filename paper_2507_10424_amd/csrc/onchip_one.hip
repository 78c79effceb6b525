// On-chip decoder kernels with one frame slot, for small batches.
#include "onchip_kernel.h"

namespace ldpc {
namespace onchip {
#define LDPC_ONE_ROW(N)                                                                                              \
    {&k_onchip<42, 0, N>, &k_onchip<43, 0, N>, &k_onchip<44, 0, N>, &k_onchip<45, 0, N>, &k_onchip<46, 0, N>,         \
     &k_onchip<47, 0, N>, &k_onchip<48, 0, N>, &k_onchip<49, 0, N>, &k_onchip<50, 0, N>, &k_onchip<51, 0, N>,         \
     &k_onchip<52, 0, N>, &k_onchip<53, 0, N>, &k_onchip<54, 0, N>, &k_onchip<55, 0, N>, &k_onchip<56, 0, N>,         \
     &k_onchip<57, 0, N>}
const KernelFn kKernelsOne[2][kNumKernels - kNumVariants] = {LDPC_ONE_ROW(false), LDPC_ONE_ROW(true)};
} // namespace onchip
} // namespace ldpc
