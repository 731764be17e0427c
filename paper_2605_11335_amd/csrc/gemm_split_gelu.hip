// The linear-layer kernels with the split gelu epilogue, in a translation unit of their own (they compile in parallel).
#include "gemm_kernel.h"

hipError_t gemm_launch_split_gelu(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    return launch_tile<EPI_SPLIT_GELU>(tile, g, second, s);
}
