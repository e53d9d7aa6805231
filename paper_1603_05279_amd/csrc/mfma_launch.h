// Host side shared by the sources that instantiate the matrix-core convolution kernel (conv_mfma_kernel.h), one source per
// group of operand formats so that they compile side by side.
#pragma once
#include "xnor_internal.h"

namespace xnor {

// Tiling override and LDS budget of xnor_set_tuning (0 = the library's choice of tiling).
int mfma_tile_override();
int mfma_lds_budget();

// One convolution with operand format FMT: 0 int8 signs, 1 4-bit signs, 2 digits of real inputs, 3 int8 levels, 4 bfloat16 parts, 5 levels
// of at most two bits as 4-bit floats, 6 bfloat16 parts made of digits.  last: no other form follows where this one refuses the geometry.
template <int FMT>
xnor_status launch_fmt(const uint32_t *xbits, const void *wimg, const float *K, const float *A, const float *alpha, float *out,
                       int32_t *dot_out, const ConvGeom &g, hipStream_t stream, const FuseArgs *fz, bool last = false);

// Matrix instructions per 64 channels and 32 x 32 results that digits take less than parts: 5 for 64 channels of a tap, 3 for 16.
inline long long bwn_digits_save(const ConvGeom &g) { return (long long)g.taps * (3 * ((g.c + 15) / 16) - 5 * ((g.cw + 1) / 2)); }

// A_next[m] = (part[0][m] + part[1][m] + ...) / k_out, planes added in order: second launch of the fused epilogue when the
// filters span several workgroups
xnor_status launch_sum_planes(const float *part, float *A_next, int m_total, int planes, float k_out, hipStream_t stream);

}  // namespace xnor
