// Binary gradient (sec. 3.2, paragraph "Binary Gradient"): the gradient that meets the weight filters in
// the backward convolution is binarised like the forward input, with the largest magnitude of the tensor
// as its scaling factor.  The forward layer is out = dot * K * alpha_k, so that gradient is
// gd = (g_out * alpha_k) * K; this file produces its sign words (packed over the filters, the channel
// axis of the backward convolution) and max |gd| per image.  The convolution itself is the forward
// kernel run on the transposed, 180-degree-rotated filters (pack_weights.hip, TRANSPOSED).
#include "xnor_internal.h"
#include <algorithm>
#include <cmath>

namespace xnor {

// Much the forward BinActiv kernel's work split: one workgroup = one or several times 64 consecutive pixels of one image x
// all filters, lanes along the pixels (contiguous in NCHW), the NW waves share the filters in groups of 8
// (one byte of a packed word), words assembled in LDS and written as one contiguous run.  The maximum
// is reduced over the waves in LDS, over the last wave by lane exchanges, and merged into gmax[image] with an
// integer atomic maximum on the float's bit pattern (|gd| >= 0, so the patterns order like the values;
// the result does not depend on the order of arrival; NaN magnitudes are ignored).
// What bounds it: memory.  Eight waves from 57 filters on (a group of filters each at least), masks only in a last group that lacks
// filters, one wave's lane exchanges and one atomic per workgroup, which takes several tiles where that pays (bingrad_run).
// Against four waves and an atomic per tile, us in a graph with the launch that clears gmax: 256 of 64x56x56 51.8 -> 33.6, 256 of 128x28x28
// 22.7 -> 19.9, 128 of 384x13x13 12.9 -> 9.5, 256 of 512x7x7 12.1 -> 7.7, 200 of 17x31x31 12.6 -> 7.8, 9 of 147x29x23 6.85 -> 5.8.
template <bool HAS_ALPHA, bool HAS_K, int NW>
__global__ __launch_bounds__(64 * NW) void bingrad_binarize_kernel(
    const float *__restrict__ g, const float *__restrict__ K, const float *__restrict__ alpha,
    uint32_t *__restrict__ gbits, float *__restrict__ gmax, int c, int hw, int cw, int run, int parts_per_image)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    float(*part)[64] = reinterpret_cast<float(*)[64]>(smem);            // [NW][64]
    uint8_t *wbytes = smem + NW * 64 * sizeof(float);                   // [run * 64 px][cw words][4 bytes]
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // workgroups go to the 8 XCDs round-robin; within every complete window of 64 tiles each XCD takes a
    // run of 8 consecutive ones, so the cache lines that straddle tile boundaries hit in its own L2
    const unsigned b = blockIdx.x, win = (b >> 6) << 6;
    const int blk = (int)(win + 64u <= gridDim.x ? win + ((b & 7u) << 3) + ((b >> 3) & 7u) : b);
    const int img = blk / parts_per_image;
    const int p0 = (blk - img * parts_per_image) * run * 64, npx = min(run * 64, hw - p0);
    const float *gi = g + (size_t)img * c * hw;
    const float *Ki = HAS_K ? K + (size_t)img * hw : nullptr;
    const int groups = (c + 7) >> 3, turns = (groups + NW - 1) / NW;    // (a wave without a group left repeats the last one)
    float m = 0.0f;
    int turn = 0, t0 = 0;                                               // turn of the waves over the filters, first pixel of the 64
    const int steps = turns * ((npx + 63) >> 6);
#pragma unroll 4
    for (int step = 0; step < steps; ++step) {
        const int gidx = min(wave + NW * turn, groups - 1), ch0 = gidx * 8;
        const int pc = min(p0 + t0 + lane, hw - 1);                     // (lanes past the image repeat its last pixel, which changes no maximum)
        const float kp = HAS_K ? Ki[pc] : 1.0f;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = gi[(size_t)min(ch0 + j, c - 1) * hw + pc];
        uint32_t byte = 0;
        auto signs = [&](int real) {                                    // filters of the group that exist
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (j >= real) break;
                float gd = v[j];
                if (HAS_ALPHA) gd = gd * alpha[ch0 + j];
                if (HAS_K) gd = gd * kp;
                byte |= gd >= 0.0f ? 1u << j : 0u;
                const float a = __builtin_fabsf(gd);
                m = a > m ? a : m;
            }
        };
        if (ch0 + 8 <= c) signs(8);
        else signs(c - ch0);
        wbytes[(size_t)((t0 + lane) * cw) * 4 + gidx] = (uint8_t)byte;
        if (++turn == turns) {
            turn = 0;
            t0 += 64;
        }
    }
    part[wave][lane] = m;
    __syncthreads();
    if (wave == NW - 1) {                 // one wave reduces, the others write the words
#pragma unroll
        for (int q = 0; q < NW - 1; ++q) m = part[q][lane] > m ? part[q][lane] : m;
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) {
            const float o = __shfl_xor(m, s, 64);
            m = o > m ? o : m;
        }
        if (lane == 0) atomicMax(reinterpret_cast<unsigned int *>(gmax + img), __float_as_uint(m));
    }
    const uint32_t *wsrc = reinterpret_cast<const uint32_t *>(wbytes);
    uint32_t *dst = gbits + ((size_t)img * hw + p0) * cw;
    const int nwords = npx * cw;
    const int tail_bytes = cw * 4 - groups;          // bytes of the last word no group wrote
    const uint32_t tail_mask = 0xFFFFFFFFu >> (8 * tail_bytes);
    for (int i = tid; i < nwords; i += 64 * NW) {
        uint32_t word = wsrc[i];
        if (i % cw == cw - 1) word &= tail_mask;
        dst[i] = word;
    }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float *__restrict__ p, int count)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0.0f;
}

__global__ __launch_bounds__(256) void bingrad_plane_kernel(const float *__restrict__ gmax,
                                                            float *__restrict__ plane, int hw)
{
    const float m = gmax[blockIdx.y];
    for (int i = blockIdx.x * 256 + threadIdx.x; i < hw; i += gridDim.x * 256)
        plane[(size_t)blockIdx.y * hw + i] = m;
}

// Tiles of 64 pixels per workgroup of bingrad_binarize_kernel: a run of up to 8 of an image.  A tile of its own costs an atomic maximum each, about 5 ns
// and 400 ns / n, since all of them meet in the few cache lines of gmax (64 of 64x56x56, 3136 tiles 27.5 us, runs of 8 13.5; 30 of 128x56x56 19.8
// and 13.4 with runs of 4; 256 of 64x56x56 53.6 and 34.5); long runs leave the CUs of a last or only round with unequal shares of the memory's
// 5.5 TB/s (146 of 448x27x27, 1752 workgroups of one tile 34.4, 292 of six 48.5; 256 of 256x20x20 from memory 24.9 and 30), and less than two workgroups per CU
// do not keep it busy.  The run whose slower side is the shortest: 280 layers, 1.02 of the best run's time in the mean (one tile each 1.11, two
// 1.11, the longest run that leaves every CU a workgroup 1.06).
static int bingrad_run(int n, int k_out, int hw, size_t words, int waves)
{
    const int tiles = (hw + 63) / 64, longest = (int)std::min<long long>({8, tiles, (long long)(32 * 1024 / words)});
    const double memory = (double)n * k_out * hw * 4 / 5.5e6, atomic = 0.005 + 0.4 / n, round = 256.0 * (32 / waves);      // us; workgroups
    double best = 0;
    int best_run = 1;
    for (int run = 1; run <= longest; ++run) {
        const double blocks = (double)n * ((tiles + run - 1) / run), share = blocks / 256;
        const double uneven = (blocks <= round ? std::ceil(share) / share : 1.0) * std::max(2.0 / share, 1.0);
        const double cost = std::max(memory * uneven, blocks * atomic);
        if (run == 1 || cost < best) {
            best = cost;
            best_run = run;
        }
    }
    return best_run;
}

xnor_status launch_bingrad_binarize(const float *g, const float *K, const float *alpha, uint32_t *gbits,
                                    float *gmax, int n, int k_out, int hw, hipStream_t stream)
{
    const int cw = (k_out + 31) / 32;
    const int tiles = (hw + 63) / 64;
    const bool wide = k_out > 56;               // a group of 8 filters for each of eight waves
    const size_t words = (size_t)64 * cw * 4;
    long long run = bingrad_run(n, k_out, hw, words, wide ? 8 : 4);
    const int parts = (int)((tiles + run - 1) / run);
    run = (tiles + parts - 1) / parts;
    const size_t lds = (wide ? 8 : 4) * 64 * sizeof(float) + words * run;
    if (words + 16 > 64 * 1024 || (long long)n * tiles > 0x7fffffffLL) return XNOR_ERR_UNSUPPORTED;
    // the maxima start at zero: cleared by a kernel, so that the sequence can be captured in a graph
    fill_zero_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(gmax, n);
    const dim3 grid((unsigned)(n * parts));
    // (nearly 8160 filters: the words and the waves' maxima pass the default limit of dynamic LDS together)
#define XNOR_BG_NW(HA, HK, NW)                                                                                                   \
    do {                                                                                                                         \
        auto kern = bingrad_binarize_kernel<HA, HK, NW>;                                                                         \
        if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, \
                                                   80 * 1024) != hipSuccess)                                                     \
            return XNOR_ERR_HIP;                                                                                                 \
        kern<<<grid, dim3(64 * NW), lds, stream>>>(g, K, alpha, gbits, gmax, k_out, hw, cw, (int)run, parts);                              \
    } while (0)
#define XNOR_BG(HA, HK) do { if (wide) XNOR_BG_NW(HA, HK, 8); else XNOR_BG_NW(HA, HK, 4); } while (0)
    if (alpha) { if (K) XNOR_BG(true, true); else XNOR_BG(true, false); }
    else       { if (K) XNOR_BG(false, true); else XNOR_BG(false, false); }
#undef XNOR_BG
#undef XNOR_BG_NW
    return hip_status(hipGetLastError());
}

xnor_status launch_bingrad_scale_plane(const float *gmax, float *plane, int n, int hw, hipStream_t stream)
{
    if (n > 65535) return XNOR_ERR_UNSUPPORTED;
    const int bx = std::min((hw + 255) / 256, 64);
    bingrad_plane_kernel<<<dim3((unsigned)bx, (unsigned)n), dim3(256), 0, stream>>>(gmax, plane, hw);
    return hip_status(hipGetLastError());
}

}  // namespace xnor
