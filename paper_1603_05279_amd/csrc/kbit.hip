// k-bit quantisation (sec. 3.2, paragraph "k-bit Quantization"): q_k(x) = 2*([(2^k - 1)(x + 1)/2]/(2^k - 1) - 1/2)
// in place of sign().  With L = 2^k - 1 and the level index u = [L (x + 1)/2], q_k = (2u - L)/L: an odd integer
// in [-L, L] over L.  The convolution of ka-bit inputs with kw-bit weights is therefore an integer contraction
// of the numerators divided by La*Lw, and runs as ONE int8 matrix-core convolution (conv_mfma_kernel.h, operand
// format 3: int32 accumulation, exact) on the numerators stored as int8; zero padding stays exact.
// (The same sum could be formed from ka*kw binary convolutions of the bit planes, q_k = sum_p 2^p s_p / L; on
// this chip the int8 contraction is ka*kw times less matrix work at half the 4-bit rate.)
#include "xnor_internal.h"
#include <type_traits>

namespace xnor {

// Level indices u of four inputs, one per byte: u = floor(((x + 1) * 0.5) * L + 0.5), x clamped to [-1, 1] (NaN -> -1), each operation
// rounded to float in this order (contraction is disabled for the build): the float value decides the level.  Rounding keeps order, so x + 1 is
// clamped instead, to [0, 2]: the addition quiets a signaling NaN, which the median of three would answer with 2.  Halving is exact, so
// (x + 1) * (L / 2) is the same float; the value lies in [0.5, L + 0.5], where conversion to integer is the floor and stays within 0 .. L.
// One bit: the comparison of the sign rule (x + 1 rounds to 1 for -2^-25 < x < 0, which would give +1).
template <bool ONE_BIT> __device__ __forceinline__ uint32_t qk_indices(const float *x, float half_L)
{
    uint32_t u = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t q = ONE_BIT ? (x[i] >= 0.0f ? 1u : 0u)
                                   : (uint32_t)(__builtin_amdgcn_fmed3f(x[i] + 1.0f, 0.0f, 2.0f) * half_L + 0.5f);
        u |= q << (8 * i);
    }
    return u;
}

// The numerators 2u - L of four level indices (u at most 127), byte by byte: 2u with its top bit forced on is at least 128 and borrows
// nothing from its neighbour; the top bit is put right afterwards.
__device__ __forceinline__ uint32_t qk_numerators(uint32_t u, uint32_t L4)
{
    const uint32_t x = u << 1, top = 0x80808080u;
    return ((x | top) - L4) ^ (~x & top);
}

// x [n][c][hw] float -> xq [n][hw][cw][32] int8: byte j of word wd = 2u - L of channel wd*32 + j (0 past the
// last channel).  One workgroup = 64 pixels that follow each other in the batch x 8 channel words; lanes along pixels
// (every channel row is read as coalesced 256-byte segments), the 4 waves share the 32 groups of 8 channels,
// a group's 8 bytes go to LDS (row stride 8*32 + 16 bytes: neighbouring lanes fall on different banks), from
// where each pixel's words leave as one contiguous run, 16 bytes per lane.
// What bounds it: memory, 4 bytes read and 1 written per input, once the levels take few instructions (7 per input; 18 with a clamp of the index
// and bytes put together one by one).  256 images of 256x14x14: 15.8 -> 12.6 us, 128 of 100x28x28 13.1 -> 10.8, 256 of 512x7x7 9.0 -> 6.9.
constexpr int KB_WORDS = 8, KB_ROW = KB_WORDS * 32 + 16;
__global__ __launch_bounds__(256) void kbit_levels_kernel(const float *__restrict__ x, int8_t *__restrict__ xq, int c, int hw, int cw, int L,
                                                          uint32_t pixels, uint32_t tiles, FastDiv div_tiles, FastDiv div_hw)
{
    __shared__ __attribute__((aligned(16))) uint8_t stage[64 * KB_ROW];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (runs of 8 workgroups per XCD: neighbouring pixel tiles share cache lines)
    const uint32_t b = blockIdx.x, win = b >> 6 << 6;
    const uint32_t blk = win + 64u <= gridDim.x ? win + ((b & 7u) << 3) + ((b >> 3) & 7u) : b;
    const uint32_t part = div_tiles.div(blk), m0 = (blk - part * tiles) * 64u;
    const int w0 = (int)part * KB_WORDS, nwords = min(KB_WORDS, cw - w0);
    const uint32_t m = min(m0 + lane, pixels - 1u), img = div_hw.div(m);
    const float *xi = x + (size_t)img * c * hw + (m - img * (uint32_t)hw);
    const uint32_t L4 = (uint32_t)L * 0x01010101u;
    const float half_L = 0.5f * (float)L;
    auto levels = [&](auto one_bit) {
#pragma unroll 2
        for (int gidx = wave; gidx < nwords * 4; gidx += 4) {           // groups of 8 channels of this workgroup
            const int ch0 = w0 * 32 + gidx * 8, real = c - ch0;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = xi[(size_t)min(ch0 + j, c - 1) * hw];
            uint32_t lo = qk_numerators(qk_indices<one_bit.value>(v, half_L), L4);
            uint32_t hi = qk_numerators(qk_indices<one_bit.value>(v + 4, half_L), L4);
            if (real < 8) {                                             // channels past the last one: 0
                lo = real <= 0 ? 0u : real < 4 ? lo & ((1u << (8 * real)) - 1u) : lo;
                hi = real <= 4 ? 0u : hi & ((1u << (8 * (real - 4))) - 1u);
            }
            *reinterpret_cast<uint2 *>(stage + lane * KB_ROW + gidx * 8) = make_uint2(lo, hi);
        }
    };
    if (L == 1) levels(std::true_type{});
    else levels(std::false_type{});
    __syncthreads();
    const int upp = nwords * 2;                       // 16-byte units per pixel
    const int npx = (int)min(64u, pixels - m0);
    int8_t *out = xq + ((size_t)m0 * cw + w0) * 32;
    for (int i = tid; i < npx * upp; i += 256) {
        const int px = i / upp, u = i - px * upp;
        *reinterpret_cast<uint4 *>(out + (size_t)px * cw * 32 + u * 16) =
            *reinterpret_cast<const uint4 *>(stage + px * KB_ROW + u * 16);
    }
}

xnor_status launch_kbit_pack_input(const float *x, int8_t *xq, int k, int n, int c, int hw, hipStream_t stream)
{
    const int cw = (c + 31) / 32;
    const int parts = (cw + KB_WORDS - 1) / KB_WORDS;
    if (parts > 65535 || n > 65535) return XNOR_ERR_UNSUPPORTED;
    const long long pixels = (long long)n * hw, tiles = (pixels + 63) / 64;
    if (tiles * parts > 0x7fffffffLL) return XNOR_ERR_UNSUPPORTED;
    kbit_levels_kernel<<<dim3((unsigned)(tiles * parts)), dim3(256), 0, stream>>>(
        x, xq, c, hw, cw, (1 << k) - 1, (uint32_t)pixels, (uint32_t)tiles, FastDiv::make((uint32_t)tiles), FastDiv::make((uint32_t)hw));
    return hip_status(hipGetLastError());
}

}  // namespace xnor
