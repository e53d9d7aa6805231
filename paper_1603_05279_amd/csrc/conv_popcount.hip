// Binary convolution on the vector ALU (sec. 3.2): dot = n_valid - 2*bitcount(x XOR w), then the
// fused scaling by K and alpha.
//
// Lanes run along output pixels; a wave shares one filter group, so every weight word is
// wave-uniform and is fetched through the scalar path (it reaches the XOR as a scalar operand),
// while each lane holds the words of its own pixel for the current tap.  Out-of-bounds taps are
// skipped per lane, which is exactly "padding contributes 0".
#include "xnor_internal.h"
#include "linear_route.h"

namespace xnor {

template <int F, int CH>   // F filters per thread, CH channel words per inner chunk (divides cw)
__global__ __launch_bounds__(256) void conv_popcount_kernel(
    const uint32_t *__restrict__ xbits, const uint32_t *__restrict__ wbits,
    const float *__restrict__ K, const float *__restrict__ A, const float *__restrict__ alpha,
    float *__restrict__ out, int32_t *__restrict__ dot_out, ConvGeom g)
{
    const uint32_t m = blockIdx.x * 256u + threadIdx.x;
    const bool live = m < (uint32_t)g.m_total;
    const uint32_t mm = live ? m : (uint32_t)g.m_total - 1u;
    const uint32_t img = g.div_howo.div(mm);
    const uint32_t pix = mm - img * (uint32_t)(g.ho * g.wo);
    const uint32_t oy = g.div_wo.div(pix);
    const uint32_t ox = pix - oy * (uint32_t)g.wo;
    const int k0 = blockIdx.y * F;

    uint32_t acc[F];
#pragma unroll
    for (int f = 0; f < F; ++f) acc[f] = 0;
    int valid_taps = 0;

    for (int dy = 0; dy < g.kh; ++dy) {
        const int iy = (int)oy * g.sh - g.ph + dy;
        for (int dx = 0; dx < g.kw; ++dx) {
            const int ix = (int)ox * g.sw - g.pw + dx;
            const bool ok = live && iy >= 0 && iy < g.h && ix >= 0 && ix < g.w;
            if (!ok) continue;
            ++valid_taps;
            const int t = dy * g.kw + dx;
            const uint32_t *xp = xbits + (((size_t)img * g.h + iy) * g.w + ix) * g.cw;
            for (int w0 = 0; w0 < g.cw; w0 += CH) {
                uint32_t a[CH];
#pragma unroll
                for (int i = 0; i < CH; ++i) a[i] = xp[w0 + i];
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const int k = min(k0 + f, g.k_out - 1);
                    const uint32_t *wp = wbits + ((size_t)k * g.taps + t) * g.cw + w0;
#pragma unroll
                    for (int i = 0; i < CH; ++i) acc[f] += __builtin_popcount(a[i] ^ wp[i]);
                }
            }
        }
    }
    if (!live) return;
    const int n_valid = g.c * valid_taps;
    const float Km = K ? K[m] : box_K(A, g, m);
    const size_t plane = (size_t)g.ho * g.wo;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int k = k0 + f;
        if (k < g.k_out) {
            const int dot = n_valid - 2 * (int)acc[f];
            const size_t o = ((size_t)img * g.k_out + k) * plane + pix;
            out[o] = (float)dot * Km * alpha[k];
            if (dot_out) dot_out[o] = dot;
        }
    }
}

// Same loop over weights in scalar-path order: for one (tap, channel word) the 32 filters' words are
// one aligned 128-byte run, fetched with wide scalar loads that overlap the vector work, instead of
// one dependent scalar load per filter.
template <int CH>   // channel words per inner chunk (divides cw)
__global__ __launch_bounds__(256) void conv_popcount_t_kernel(
    const uint32_t *__restrict__ xbits, const uint32_t *__restrict__ wpop,
    const float *__restrict__ K, const float *__restrict__ A, const float *__restrict__ alpha,
    float *__restrict__ out, int32_t *__restrict__ dot_out, ConvGeom g)
{
    constexpr int F = 32;
    const uint32_t m = blockIdx.x * 256u + threadIdx.x;
    const bool live = m < (uint32_t)g.m_total;
    const uint32_t mm = live ? m : (uint32_t)g.m_total - 1u;
    const uint32_t img = g.div_howo.div(mm);
    const uint32_t pix = mm - img * (uint32_t)(g.ho * g.wo);
    const uint32_t oy = g.div_wo.div(pix);
    const uint32_t ox = pix - oy * (uint32_t)g.wo;
    const int kb = blockIdx.y;
    const uint32_t *wblk = wpop + (size_t)kb * g.taps * g.cw * 32;

    uint32_t acc[F];
#pragma unroll
    for (int f = 0; f < F; ++f) acc[f] = 0;
    int valid_taps = 0;
    for (int dy = 0; dy < g.kh; ++dy) {
        const int iy = (int)oy * g.sh - g.ph + dy;
        for (int dx = 0; dx < g.kw; ++dx) {
            const int ix = (int)ox * g.sw - g.pw + dx;
            const bool ok = live && iy >= 0 && iy < g.h && ix >= 0 && ix < g.w;
            if (!ok) continue;
            ++valid_taps;
            const int t = dy * g.kw + dx;
            const uint32_t *xp = xbits + (((size_t)img * g.h + iy) * g.w + ix) * g.cw;
            const uint32_t *wt = wblk + (size_t)t * g.cw * 32;
            for (int w0 = 0; w0 < g.cw; w0 += CH) {
                uint32_t a[CH];
#pragma unroll
                for (int i = 0; i < CH; ++i) a[i] = xp[w0 + i];
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const uint32_t *wr = wt + (size_t)(w0 + i) * 32;
#pragma unroll
                    for (int f = 0; f < F; ++f) acc[f] += __builtin_popcount(a[i] ^ wr[f]);
                }
            }
        }
    }
    if (!live) return;
    const int n_valid = g.c * valid_taps;
    const float Km = K ? K[m] : box_K(A, g, m);
    const size_t plane = (size_t)g.ho * g.wo;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int k = kb * F + f;
        if (k < g.k_out) {
            const int dot = n_valid - 2 * (int)acc[f];
            const size_t o = ((size_t)img * g.k_out + k) * plane + pix;
            out[o] = (float)dot * Km * alpha[k];
            if (dot_out) dot_out[o] = dot;
        }
    }
}

template <int F>
static xnor_status launch_f(const uint32_t *xbits, const uint32_t *wbits, const float *K, const float *A,
                            const float *alpha, float *out, int32_t *dot_out, const ConvGeom &g,
                            hipStream_t stream)
{
    dim3 grid((unsigned)((g.m_total + 255) / 256), (unsigned)((g.k_out + F - 1) / F)), block(256);
    if (grid.y > 65535u) return XNOR_ERR_UNSUPPORTED;
#define XNOR_GO(CH) conv_popcount_kernel<F, CH><<<grid, block, 0, stream>>>(xbits, wbits, K, A, alpha, out, dot_out, g)
    if (g.cw % 8 == 0) XNOR_GO(8);
    else if (g.cw % 4 == 0) XNOR_GO(4);
    else if (g.cw % 3 == 0) XNOR_GO(3);
    else if (g.cw % 2 == 0) XNOR_GO(2);
    else XNOR_GO(1);
#undef XNOR_GO
    return hip_status(hipGetLastError());
}

xnor_status launch_conv_popcount(const uint32_t *xbits, const uint32_t *wbits, const void *wmfma, const float *K,
                                 const float *A, const float *alpha, float *out, int32_t *dot_out,
                                 const ConvGeom &g, hipStream_t stream)
{
    if (wmfma) {
        const uint32_t *wpop = reinterpret_cast<const uint32_t *>(
            static_cast<const uint8_t *>(wmfma) + wimg_i8_bytes(g.k_out, g.c, g.taps) + wimg_f4_bytes(g.k_out, g.c, g.taps));
        dim3 grid((unsigned)((g.m_total + 255) / 256), (unsigned)g.fblocks), block(256);
        if (grid.y > 65535u) return XNOR_ERR_UNSUPPORTED;
#define XNOR_GO(CH) conv_popcount_t_kernel<CH><<<grid, block, 0, stream>>>(xbits, wpop, K, A, alpha, out, dot_out, g)
        if (g.cw % 2 == 0) XNOR_GO(2);
        else XNOR_GO(1);
#undef XNOR_GO
        return hip_status(hipGetLastError());
    }
    return launch_f<32>(xbits, wbits, K, A, alpha, out, dot_out, g, stream);
}

// Fully connected layers whose batch is small: every pair of rows reads the weights once (from memory the first, from L2
// the others), so the time is that of bringing them in.  The matrix-core form reads them as 4-bit operands (four times the
// packed bits) and walks the whole K in one workgroup; here 16 lanes share a filter's row of packed words, V words per
// lane and load with U loads in flight, each word meeting the same word of NB rows of the batch.  The 16 partial counts
// meet by lane exchanges.  Bound by the latency of one trip to memory and the launch.  9216 -> 4096, launches of one graph:
// one row 9.4 -> 2.1 us, eight rows 11.0 -> 3.6 us.  (Two rows per workgroup: with four or eight the rows' counts are a
// serial chain in one wave, 0.6 and 3.1 us more for eight rows.)  A lane's loads past the end of a row fetch its first words again and
// count nothing: 2048 rows x 16 filters take 4.2 us at any length from 512 to 9216 features, 7.8 us at 25088 (three passes).
constexpr int FC_LANES = 16;
template <int V, int NB>
__global__ __launch_bounds__(256) void linear_popcount_kernel(
    const uint32_t *__restrict__ xbits, const uint32_t *__restrict__ wbits, const float *__restrict__ Krow,
    const float *__restrict__ alpha, float *__restrict__ out, int32_t *__restrict__ dot_out, int n, int c, int cw,
    int k_out)
{
    constexpr int U = V == 4 ? 5 : 8;                  // loads in flight per lane (linear_words_per_pass in all)
    static_assert(FC_LANES * V * U == linear_words_per_pass(V), "the rule counts passes of this size");
    typedef uint32_t vec __attribute__((ext_vector_type(V)));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane & (FC_LANES - 1);
    const int f = (blockIdx.x * 4 + wave) * (64 / FC_LANES) + lane / FC_LANES;
    const int n0 = blockIdx.y * NB;
    const uint32_t *wr = wbits + (size_t)min(f, k_out - 1) * cw;
    uint32_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = 0;
    for (int base = 0; base < cw; base += FC_LANES * V * U) {
        vec w[U];
        int idx[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + (u * FC_LANES + sub) * V;      // V divides cw: a lane's V words lie in the row or none does
            ok[u] = i < cw;
            idx[u] = ok[u] ? i : 0;
            w[u] = *reinterpret_cast<const vec *>(wr + idx[u]);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint32_t *xr = xbits + (size_t)min(n0 + b, n - 1) * cw;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const vec x = *reinterpret_cast<const vec *>(xr + idx[u]);
                uint32_t cnt = 0;
#pragma unroll
                for (int q = 0; q < V; ++q) cnt += __builtin_popcount(x[q] ^ w[u][q]);
                acc[b] += ok[u] ? cnt : 0u;
            }
        }
    }
    uint32_t mine = 0;                                 // lane b of the 16 keeps the count of row n0 + b
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        uint32_t s = acc[b];
#pragma unroll
        for (int off = FC_LANES / 2; off > 0; off >>= 1) s += (uint32_t)__shfl_xor((int)s, off, 64);
        mine = sub == b ? s : mine;
    }
    const int m = n0 + sub;
    if (sub < NB && m < n && f < k_out) {
        const int dot = c - 2 * (int)mine;
        const size_t o = (size_t)m * k_out + f;
        out[o] = (float)dot * Krow[m] * alpha[f];
        if (dot_out) dot_out[o] = dot;
    }
}

bool linear_popcount_applies(const ConvGeom &g, bool matrix_image)
{
    if (g.h != 1 || g.w != 1 || g.taps != 1 || g.ph != 0 || g.pw != 0 || g.dil_h != 1 || g.dil_w != 1) return false;
    if (matrix_image && linear_words_applies(g)) return linear_few_rows_ahead_of_words(g.n, g.k_out, g.c, g.cw);
    return linear_popcount_route(g.n, g.k_out, g.c, g.cw, matrix_image);
}

// (a 1x1 image and filter: K of a row is its A)
xnor_status launch_linear_popcount(const uint32_t *xbits, const uint32_t *wbits, const float *Krow, const float *alpha,
                                   float *out, int32_t *dot_out, const ConvGeom &g, hipStream_t stream)
{
    constexpr int FPB = 4 * 64 / FC_LANES;             // filters per workgroup
    const unsigned gx = (unsigned)((g.k_out + FPB - 1) / FPB);
#define XNOR_GO(V, NB)                                                                                                 \
    linear_popcount_kernel<V, NB><<<dim3(gx, (unsigned)((g.n + NB - 1) / NB)), dim3(256), 0, stream>>>(                \
        xbits, wbits, Krow, alpha, out, dot_out, g.n, g.c, g.cw, g.k_out)
#define XNOR_GO_N(V)                                                                                                   \
    do { if (g.n == 1) XNOR_GO(V, 1); else XNOR_GO(V, 2); } while (0)
    switch (linear_words_per_load(g.cw)) {
    case 4: XNOR_GO_N(4); break;
    case 2: XNOR_GO_N(2); break;
    default: XNOR_GO_N(1);
    }
#undef XNOR_GO_N
#undef XNOR_GO
    return hip_status(hipGetLastError());
}

}  // namespace xnor
