// Max-pooling in the convolution's epilogue (4-bit operands).
#include "conv_mfma_kernel.h"

namespace xnor {

// Pooled-epilogue launch of one tiling (4-bit operands): a pixel tile is a group of pooled rows of one image.
template <int FW, int PW, int WF, int WP>
static xnor_status launch_cfg_pool(const uint32_t *xbits, const void *wimg, const float *K, const float *A,
                                   const float *alpha, float *out_pool, const ConvGeom &g, const PoolPlan &pool,
                                   hipStream_t stream)
{
    constexpr int FT = 32 * FW * WF, PT = 32 * PW * WP, WAVES = WF * WP;
    MfmaPlan pl;
    const int conv_rows = (pool.pr - 1) * pool.sh + pool.ph;          // convolution rows under a tile
    if (conv_rows * g.wo > PT) return XNOR_ERR_UNSUPPORTED;
    if (!make_plan(g, PT, 1, mfma_lds_budget(), 0, FT * 4, &pl, (conv_rows - 1) * g.sh + g.kh)) return XNOR_ERR_UNSUPPORTED;
    size_t lds = plan_lds_bytes(pl, 1, g.wp, PT, 0, FT * 4);
    pl.lut_offset = plan_lut_offset(pl, 1, g.wp, PT, 0, FT * 4);
    lds = std::max(lds, (size_t)WAVES * 16 * (PT + 1) * sizeof(float));       // the epilogue's per-wave y tiles
    if (lds > (size_t)LDS_LIMIT) return XNOR_ERR_UNSUPPORTED;
    set_direct_staging(&pl, g, 1, PT);
    const int build = pl.vec == 0 ? 0 : pl.cc_words == g.cw ? 1 : 2;
    auto kern = build == 1   ? conv_mfma_kernel<1, FW, PW, WF, WP, false, true, true>
                : build == 2 ? conv_mfma_kernel<1, FW, PW, WF, WP, false, false, true, 1, true>
                             : conv_mfma_kernel<1, FW, PW, WF, WP, false, false, true>;
    static std::atomic<bool> attr_done[3];
    if (xnor_status s = allow_full_lds(kern, attr_done[build])) return s;
    const long long ptiles = (long long)g.n * pool.groups;
    if (ptiles > 0x7fffffffLL) return XNOR_ERR_UNSUPPORTED;
    pl.ptiles = (int)ptiles;
    pl.ftiles = (g.k_out + FT - 1) / FT;
    pl.wmajor = 0;
    pl.stream_out = 0;
    pl.pool = pool;
    if (pl.ftiles > 65535) return XNOR_ERR_UNSUPPORTED;
    const size_t img_bytes = wimg_pop_bytes(g.k_out, g.c, g.taps);
    if (img_bytes > 0x7fffffffull) return XNOR_ERR_UNSUPPORTED;
    // the XCD-aware tile order works on whole windows of 64 pixel tiles; the grid is not padded beyond ptiles
    kern<<<dim3((unsigned)pl.ptiles, (unsigned)pl.ftiles), dim3(64 * WAVES), lds, stream>>>(
        ConvArgs{xbits, reinterpret_cast<const v4i *>(wimg), K, A, alpha, out_pool, nullptr, (uint32_t)img_bytes, g, pl,
                 FuseArgs{}});
    return hip_status(hipGetLastError());
}

xnor_status launch_conv_mfma_pool(const uint32_t *xbits, const void *wmfma, const float *K, const float *A,
                                  const float *alpha, float *out_pool, const ConvGeom &g, int ph, int pw, int sh,
                                  int sw, int relu, hipStream_t stream)
{
    if ((long long)g.c * g.taps >= (1ll << 24)) return XNOR_ERR_UNSUPPORTED;       // exact float accumulation
    PoolPlan pool;
    pool.ph = ph; pool.pw = pw; pool.sh = sh; pool.sw = sw; pool.relu = relu;
    pool.hpo = (g.ho - ph) / sh + 1;
    pool.wpo = (g.wo - pw) / sw + 1;
    pool.div_wpo = FastDiv::make((uint32_t)pool.wpo);
    // Tile: 256 filters x 96, 160 or 192 pixels.  Each holds as many pooled rows as its pixels allow; the
    // choice minimises (rounds of workgroups over the CUs' workgroup slots) x (pixels per tile), the smaller
    // tile on a tie.
    const int pts[3] = {96, 160, 192};
    int best = -1, best_pr = 0;
    long long best_cost = 0;
    const int ftiles = (g.k_out + 255) / 256;
    for (int t = 0; t < 3; ++t) {
        const int rows_fit = pts[t] / g.wo;                     // convolution rows a tile can hold
        if (rows_fit < ph) continue;
        const int pr = std::min((rows_fit - ph) / sh + 1, pool.hpo);
        const long long groups = (pool.hpo + pr - 1) / pr;
        const long long wgs = (long long)g.n * groups * ftiles;
        const long long slots = t == 0 ? 512 : 256;            // two workgroups of the 96-pixel tile share a CU
        const long long cost = (wgs + slots - 1) / slots * pts[t];
        if (best < 0 || cost < best_cost) { best = t; best_cost = cost; best_pr = pr; }
    }
    if (best < 0) return XNOR_ERR_UNSUPPORTED;                  // a pooling window's rows do not fit any tile
    pool.pr = best_pr;
    pool.groups = (pool.hpo + best_pr - 1) / best_pr;
    pool.div_groups = FastDiv::make((uint32_t)pool.groups);
    const uint8_t *img = static_cast<const uint8_t *>(wmfma) + wimg_i8_bytes(g.k_out, g.c, g.taps) +
                         wimg_f4_bytes(g.k_out, g.c, g.taps);
    switch (best) {
    case 0: return launch_cfg_pool<2, 3, 4, 1>(xbits, img, K, A, alpha, out_pool, g, pool, stream);
    case 1: return launch_cfg_pool<2, 5, 4, 1>(xbits, img, K, A, alpha, out_pool, g, pool, stream);
    default: return launch_cfg_pool<2, 6, 4, 1>(xbits, img, K, A, alpha, out_pool, g, pool, stream);
    }
}

}  // namespace xnor
