// The epilogue whose plain features are heads of q, k and v, placed as attention reads them, the others through the erf form of GELU (gemm_kernel.h).
#include "gemm_kernel.h"

hipError_t gemm_launch_heads_erf(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    return launch_tile<EPI_HEADS_ERF>(tile, g, second, s);
}
