// Prints workgroups_per_cu (csrc/ldpc_internal.h) for 1 to 16 wavefronts, one
// line per wavefronts that a SIMD holds, given on the command line; "most" is
// what dividing all waves by a workgroup's gives.
#include <cstdio>
#include <cstdlib>

#include "ldpc_internal.h"

int main(int argc, char **argv) {
    for (int a = 1; a < argc; ++a) {
        const int per_simd = std::atoi(argv[a]);
        for (int w = 1; w <= 16; ++w) std::printf("%d ", ldpc::workgroups_per_cu(w, per_simd, 4 * per_simd / w));
        std::printf("\n");
    }
    return 0;
}
