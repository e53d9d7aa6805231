// Binary-Weight-Network convolution: digits of the real inputs, as the split wrote them or made of its bfloat16 parts, or the parts as they are.
#include "conv_mfma_kernel.h"

namespace xnor {

template xnor_status launch_fmt<2>(const uint32_t *, const void *, const float *, const float *, const float *, float *,
                                   int32_t *, const ConvGeom &, hipStream_t, const FuseArgs *, bool);
template xnor_status launch_fmt<6>(const uint32_t *, const void *, const float *, const float *, const float *, float *,
                                   int32_t *, const ConvGeom &, hipStream_t, const FuseArgs *, bool);
template xnor_status launch_fmt<4>(const uint32_t *, const void *, const float *, const float *, const float *, float *,
                                   int32_t *, const ConvGeom &, hipStream_t, const FuseArgs *, bool);

xnor_status launch_bwn_conv(const void *parts, const void *wimg, const float *alpha, float *out, const ConvGeom &g,
                            const ConvGeom &gp, hipStream_t stream)
{
    const uint32_t *x = static_cast<const uint32_t *>(parts);
    const uint8_t *words = static_cast<const uint8_t *>(wimg) + wimg_bf16_bytes(g.k_out, (g.c + 15) / 16, g.taps);
    if (bwn_in_digits(g.c)) {
        const xnor_status s = launch_fmt<2>(x, words, nullptr, nullptr, alpha, out, nullptr, g, stream, nullptr, true);
        if (s != XNOR_ERR_UNSUPPORTED) return s;
        // (rows of which not even one word's digits, 144 bytes a pixel, fit beside the smallest tile, and one group's parts, 112, do)
        return launch_fmt<6>(x, wimg, nullptr, nullptr, alpha, out, nullptr, gp, stream, nullptr);
    }
    // Up to 32 channels the digits are made while a tile is staged: that costs a wave about 1.2 us per 64 words, and every tap multiplies
    // them with 5 instructions instead of 12.  Digits win from 5 x 5 filters on, and from 3 x 3 where there are workgroups enough to
    // convert under each other's matrix instructions (bfloat16 parts against digits: 88 of 32x18x43, 5x5 -> 32 35.9 / 25.3), while they
    // take fewer instructions: up to 16 channels they do not (142 of 16 x 8 x 17, 3 x 3 -> 396, 14.0 -> 26.7; 9 of 9 x 54 x 54, 7 x 7
    // stride 2 -> 182, 7.6 -> 11.2).  A tile of its own may still decide for the parts (launch_cfg).
    const long long wgs = (long long)((g.m_total + 127) / 128) * ((g.k_out + 127) / 128);
    const bool digits = g.taps >= 25 || (g.taps >= 9 && wgs >= 128);
    if (digits && bwn_digits_save(g) > 0) {
        const xnor_status s = launch_fmt<2>(x, words, nullptr, nullptr, alpha, out, nullptr, g, stream, nullptr);
        if (s != XNOR_ERR_UNSUPPORTED) return s;
    }
    // (each form's LDS image fits where the other's does not)
    const xnor_status s = launch_fmt<4>(x, wimg, nullptr, nullptr, alpha, out, nullptr, gp, stream, nullptr);
    if (s != XNOR_ERR_UNSUPPORTED || !digits) return s;
    return launch_fmt<2>(x, words, nullptr, nullptr, alpha, out, nullptr, g, stream, nullptr, true);
}

}  // namespace xnor
