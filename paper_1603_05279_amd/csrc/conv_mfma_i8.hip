// int8 operands: signs (XNOR_ALGO_MFMA_I8) and the level numerators of k-bit tensors; those of at most two bits as 4-bit floats.
#include "conv_mfma_kernel.h"

namespace xnor {

template xnor_status launch_fmt<0>(const uint32_t *, const void *, const float *, const float *, const float *, float *,
                                   int32_t *, const ConvGeom &, hipStream_t, const FuseArgs *, bool);
template xnor_status launch_fmt<3>(const uint32_t *, const void *, const float *, const float *, const float *, float *,
                                   int32_t *, const ConvGeom &, hipStream_t, const FuseArgs *, bool);
template xnor_status launch_fmt<5>(const uint32_t *, const void *, const float *, const float *, const float *, float *,
                                   int32_t *, const ConvGeom &, hipStream_t, const FuseArgs *, bool);

}  // namespace xnor
