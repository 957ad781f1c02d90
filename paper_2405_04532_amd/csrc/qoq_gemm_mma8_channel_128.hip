// The eight-wave GEMM kernel (qoq_gemm_mma8.h) with 128 channels per tile, per-channel mode.
#include "qoq_gemm_mma8.h"

namespace qoq {

hipError_t launch_mma8_channel_128(const GemmDev& p, int mf, hipStream_t s) { return launch_mma8_tile<false, 2>(p, mf, s); }

}  // namespace qoq
