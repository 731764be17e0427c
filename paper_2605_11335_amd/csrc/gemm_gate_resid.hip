// The linear-layer kernels with the gate resid epilogue, in a translation unit of their own (they compile in parallel).
#include "gemm_kernel.h"

hipError_t gemm_launch_gate_resid(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    return launch_tile<EPI_GATE_RESID>(tile, g, second, s);
}
