// 4-bit operands (XNOR_ALGO_MFMA_F4), plain and fused epilogue.
#include "conv_mfma_kernel.h"

namespace xnor {

template xnor_status launch_fmt<1>(const uint32_t *, const void *, const float *, const float *, const float *, float *,
                                   int32_t *, const ConvGeom &, hipStream_t, const FuseArgs *, bool);

}  // namespace xnor
