// The linear-layer kernels that compute the last part of a sum cut along K and put the parts together, in a translation unit of
// their own (they compile in parallel).
#include "gemm_kernel.h"

hipError_t gemm_launch_last_part(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    return launch_tile<EPI_LAST_PART>(tile, g, second, s);
}
