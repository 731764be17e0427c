// The epilogue whose plain features are heads of q, k and v, placed as attention reads them (gemm_kernel.h).
#include "gemm_kernel.h"

hipError_t gemm_launch_heads(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    return launch_tile<EPI_HEADS>(tile, g, second, s);
}
