// The linear-layer kernels that compute the parts of a sum cut along K, in a translation unit of their own (they compile
// in parallel).
#include "gemm_kernel.h"

hipError_t gemm_launch_partial(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    return launch_tile<EPI_PARTIAL>(tile, g, second, s);
}
