// The eight-wave GEMM kernel (qoq_gemm_mma8.h) with 256 channels per tile, group mode.
#include "qoq_gemm_mma8.h"

namespace qoq {

hipError_t launch_mma8_group_256(const GemmDev& p, int mf, hipStream_t s) { return launch_mma8_tile<true, 4>(p, mf, s); }

}  // namespace qoq
