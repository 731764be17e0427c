// The linear-layer kernels whose workgroups compute the parts of a sum cut along K and put them together, in a translation unit of
// their own (they compile in parallel).
#include "gemm_kernel.h"

hipError_t gemm_launch_meet(int tile, const GemmArgs& g, const GemmArgs* second, hipStream_t s) {
    return launch_tile<EPI_MEET>(tile, g, second, s);
}
