// Host side of the matrix-core convolution (kernel: conv_mfma_kernel.h): operand format, tuning state, and the second launch
// of the fused epilogue.
#include "mfma_launch.h"
#include <atomic>

namespace xnor {

static std::atomic<int> g_tile_override{0};
static std::atomic<int> g_lds_budget{64 * 1024};
void set_mfma_tuning(int tile, int lds_budget)
{
    g_tile_override.store(tile, std::memory_order_relaxed);
    if (lds_budget > 0) g_lds_budget.store(lds_budget, std::memory_order_relaxed);
}
int mfma_tile_override() { return g_tile_override.load(std::memory_order_relaxed); }
int mfma_lds_budget() { return g_lds_budget.load(std::memory_order_relaxed); }

// second kernel of the fused epilogue when the filters span several workgroups:
// A_next[m] = (part[0][m] + part[1][m] + ...) / k_out, planes added in order
__global__ __launch_bounds__(256) void sum_planes_kernel(const float *__restrict__ part, float *__restrict__ A_next,
                                                        int m_total, int planes, float k_out)
{
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m >= m_total) return;
    float s = 0.0f;
    for (int p = 0; p < planes; ++p) s += part[(size_t)p * m_total + m];
    A_next[m] = s / k_out;
}

xnor_status launch_sum_planes(const float *part, float *A_next, int m_total, int planes, float k_out, hipStream_t stream)
{
    sum_planes_kernel<<<dim3((unsigned)((m_total + 255) / 256)), dim3(256), 0, stream>>>(part, A_next, m_total, planes, k_out);
    return hip_status(hipGetLastError());
}

xnor_status launch_conv_mfma(int fmt, const uint32_t *xbits, const void *wmfma, const float *K, const float *A,
                             const float *alpha, float *out, int32_t *dot_out,
                             const ConvGeom &g, hipStream_t stream, const FuseArgs *fz, bool last)
{
    const uint8_t *img = static_cast<const uint8_t *>(wmfma);
    // fmt 3: int8 level numerators (xbits = 32-byte words of 32 channels, wmfma = an int8 record image); no K
    // fmt 5: the same for kbit_narrow() layers, on the 4-bit record image behind it.  Three words per pixel it stages at once
    // or not at all, where int8 may take one at a time: rows too wide for that run on int8.
    if (fmt == 3 || fmt == 5) {
        if (fz) return XNOR_ERR_UNSUPPORTED;
        if (fmt == 5) {
            const xnor_status s = launch_fmt<5>(xbits, img + wimg_i8_bytes(g.k_out, g.c, g.taps), nullptr, nullptr, alpha, out,
                                                dot_out, g, stream, nullptr);
            if (s != XNOR_ERR_UNSUPPORTED) return s;
        }
        return launch_fmt<3>(xbits, img, nullptr, nullptr, alpha, out, dot_out, g, stream, nullptr);
    }
    // float accumulation of the 4-bit path is exact while every sum stays below 2^24
    if (fmt != 0 && (long long)g.c * g.taps >= (1ll << 24)) return XNOR_ERR_UNSUPPORTED;
    if (fmt == 0) return launch_fmt<0>(xbits, img, K, A, alpha, out, dot_out, g, stream, fz);
    img += wimg_i8_bytes(g.k_out, g.c, g.taps) + wimg_f4_bytes(g.k_out, g.c, g.taps);
    if (!fz && mfma_tile_override() == 0 && linear_words_applies(g)) {
        const xnor_status s = launch_linear_words(xbits, reinterpret_cast<const uint32_t *>(img), K ? K : A, alpha, out, dot_out, g, stream);
        if (s != XNOR_ERR_UNSUPPORTED) return s;
    }
    return launch_fmt<1>(xbits, img, K, A, alpha, out, dot_out, g, stream, fz, last);
}

}  // namespace xnor
