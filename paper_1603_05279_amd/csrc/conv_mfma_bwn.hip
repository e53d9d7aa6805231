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
    if (bwn_in_digits(g.c, g.w)) {
        ConvGeom gd = g;
        gd.stored_digits = 1;
        const xnor_status s = launch_fmt<2>(x, words, nullptr, nullptr, alpha, out, nullptr, gd, stream, nullptr, true);
        if (s != XNOR_ERR_UNSUPPORTED) return s;
        // (filters so tall that not even one word's digits, 144 bytes a pixel, fit beside the smallest tile, and one group's parts, 112, do)
        return launch_fmt<6>(x, wimg, nullptr, nullptr, alpha, out, nullptr, gp, stream, nullptr);
    }
    // Inputs that come as parts.  Making the digits of a word while a tile is staged costs a wave about 1.2 us per 64 words, and every tap
    // multiplies them with 5 instructions instead of 12.  Digits win from 5 x 5 filters on, and from 3 x 3 where there are workgroups enough to
    // convert under each other's matrix instructions (measured, bfloat16 parts against digits, before the split wrote digits where rows are short:
    // 128 images of 256 x 13 x 13 -> 384, 3 x 3, 102 -> 78 us; 15 of 146 x 9 x 9 -> 368, 5 x 5, 38 -> 22; 23 of 96 x 33 x 22 -> 50, 3 x 3,
    // 28.7 -> 24.8; but 6 of 288 x 23 x 20 -> 32, 3 x 3, 31 -> 35 and 21 of 264 x 11 x 11 -> 112, 1 x 1, 12.0 -> 13.5), while they take fewer
    // instructions: up to 16 channels they do not (142 of 16 x 8 x 17, 3 x 3 -> 396, 14.0 -> 26.7; 9 of 9 x 54 x 54, 7 x 7 stride 2 -> 182,
    // 7.6 -> 11.2).  A tile of its own may still decide for the parts (launch_cfg).
    const long long wgs = (long long)((g.m_total + 127) / 128) * ((g.k_out + 127) / 128);
    const bool digits = g.taps >= 25 || (g.taps >= 9 && wgs >= 128);
    if (digits && bwn_digits_save(g) > 0) {
        const xnor_status s = launch_fmt<2>(x, words, nullptr, nullptr, alpha, out, nullptr, g, stream, nullptr);
        if (s != XNOR_ERR_UNSUPPORTED) return s;
    }
    // (each form's LDS image fits where the other's does not)
    xnor_status s = launch_fmt<4>(x, wimg, nullptr, nullptr, alpha, out, nullptr, gp, stream, nullptr);
    if (s == XNOR_ERR_UNSUPPORTED && digits) s = launch_fmt<2>(x, words, nullptr, nullptr, alpha, out, nullptr, g, stream, nullptr, true);
    if (s == XNOR_ERR_UNSUPPORTED && g.c > 32) s = launch_fmt<4>(x, wimg, nullptr, nullptr, alpha, out, nullptr, gp, stream, nullptr, true);
    return s;
}

}  // namespace xnor
