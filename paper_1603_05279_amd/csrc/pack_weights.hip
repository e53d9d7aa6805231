// Weight binarisation (sec. 3.1): B = sign(W) packed to bits, alpha = ||W||_1 / n per filter.
// Runs once per layer; at inference only B and alpha are kept.  Also writes the same signs in
// matrix-core operand order, so the convolution can fetch a whole 32-filter operand as one
// contiguous KiB: once as int8 (+1/-1, 0 for channel or filter padding) for the 32x32x32 int8
// instruction and once as 4-bit floats (E2M1 0x2/0xA/0x0) for the 32x32x64 f8f6f4 instruction.
#include "mfma_common.h"
#include <type_traits>

namespace xnor {

// int8 image: for filter block fb (32 filters), tap t, channel word wd there is a 1 KiB record
// (index (fb*taps + t)*cw + wd); lane l of a wave owns bytes [16*l, 16*l+16): filter
// fb*32 + (l & 31), channels wd*32 + 16*(l >> 5) + 0..15.
// 4-bit image (after the int8 image): the (tap, word) blocks of a filter are numbered
// b = t*cw + wd and taken two per record (record fb*ceil(taps*cw/2) + b/2); lane l owns the 32
// channels of block 2*(b/2) + (l >> 5) as 32 nibbles, channel j in nibble j (low nibble first);
// a block past the end is all zero.
// MODE 1 (transposed): the filters of the data-gradient convolution of the backward pass (sec. 3.2, "Binary
// Gradient"), read straight out of the forward tensor W [c][k_out][taps] (c = forward filters, k_out =
// forward channels in this kernel's naming): filter k, channel ch, tap t is W[ch][k][taps - 1 - t], the
// forward filter rotated by 180 degrees with the two channel axes exchanged.
// MODE 3 (k-bit quantised weights as int8 levels): the int8 image alone is written, its bytes the odd-integer
// numerators 2u - L of q_aux(w) (L = 2^aux - 1) instead of +-1; wbits may be NULL; alpha[k] = `alpha_fill`
// (the caller's 1 / (La * Lw)).
// MODE 4 (at most two bits): the same, and behind the int8 image its levels as 4-bit records (Enc<5>).
// In mode 1 alpha is written as 1 (the scaling of that convolution is applied elsewhere).
__device__ __forceinline__ int qk_level_index(float x, int L)
{
    // level index u = floor(((x + 1) * 0.5) * L + 0.5) of q_k, x clamped to [-1, 1] (NaN -> -1); every
    // operation rounded to float in this order (the build disables contraction)
    float t = x >= -1.0f ? x : -1.0f;
    t = t <= 1.0f ? t : 1.0f;
    const float v = ((t + 1.0f) * 0.5f) * (float)L + 0.5f;
    if (L == 1) return x >= 0.0f ? 1 : 0;      // one bit: the sign rule's comparison, for every float
    return min(max((int)__builtin_floorf(v), 0), L);
}

// Shape of the work of one launch.  An image workgroup packs 8 filters x 32 * words channels x tap_run taps;
// workgroups of their own form alpha, one filter each (mode 0).
struct PackPlan {
    int tap_run, tap_chunks;        // taps per workgroup (at most 16), ceil(taps / tap_run)
    int words_log2, word_groups;    // channel words per workgroup (a power of two), ceil(cw / words)
    uint32_t image_groups, groups;  // image workgroups, all workgroups
    FastDiv div_tap, div_gt, div_chunks, div_wgroups, div_units;
};
constexpr int PACK_ROWS = 8;                        // filters per image workgroup: 128-byte runs of the images
constexpr int PACK_PAIRS = 16;                      // (word, tap) pairs of a workgroup at most
constexpr int PACK_BYTES = PACK_ROWS * (32 * PACK_PAIRS + 4) + 32 * 16 * 4;     // either layout below, rows padded

// What bounds it: the bytes are few (4 per weight read by the image workgroups and, in mode 0, again for alpha; 1.75
// written), so the time of a layer is round trips and instructions.  Each workgroup reads 8 filters x 32 channels x the
// taps once, as runs of memory copied without index arithmetic to one byte per weight in LDS; a wave-wide comparison of 64
// such bytes gives two packed words, and all images are written from the words: the int8 and 4-bit images in whole cache
// lines, the scalar-path image in 32-byte runs, wbits in runs of the words a workgroup holds (one word from 9 taps on).
// Measured back to back against one workgroup per filter that walked it four times: 14.2 -> 6.2 us at 128 filters of
// 128 x 3 x 3 (13.6 -> 6.4 us transposed), 292 -> 95 us at 4096 x 9216 (0.30 GB read, 0.07 GB written: 3.9 TB/s; 358 -> 264 us
// transposed, where a row of memory is a channel).
template <int MODE>
__global__ __launch_bounds__(256) void pack_weights_kernel(
    const float *__restrict__ w, uint32_t *__restrict__ wbits, float *__restrict__ alpha,
    int8_t *__restrict__ wmfma, int k_out, int c, int taps, int cw, int levels, float alpha_fill, PackPlan pl)
{
    __shared__ __attribute__((aligned(16))) uint8_t bytes[PACK_BYTES];
    __shared__ uint32_t words[PACK_PAIRS * PACK_ROWS];                           // [word * tap_run + tap][filter]
    __shared__ float red[256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (uint32_t blk = blockIdx.x; blk < pl.groups; blk += gridDim.x) {
        if (blk != blockIdx.x) __syncthreads();     // the previous turn's LDS contents are consumed
        if (MODE == 0 && blk >= pl.image_groups) {
            // alpha of one filter: strided partial sums, then a tree of fixed order
            const uint32_t k = blk - pl.image_groups;
            const size_t n = (size_t)c * taps;
            const float *wf = w + (size_t)k * n;
            float s = 0.0f;
            for (size_t i0 = tid; i0 < n; i0 += 256 * 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = i0 + u * 256 < n ? wf[i0 + u * 256] : 0.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) s += __builtin_fabsf(v[u]);          // (+0 past the end changes nothing)
            }
            red[tid] = s;
            __syncthreads();
            if (tid < 64) {
                float t = (red[tid] + red[tid + 128]) + (red[tid + 64] + red[tid + 192]);
#pragma unroll
                for (int step = 32; step > 0; step >>= 1) t += __shfl_down(t, step, 64);
                if (tid == 0) alpha[k] = t / (float)n;
            }
            continue;
        }
        const uint32_t fq = pl.div_chunks.div(blk), tchunk = blk - fq * (uint32_t)pl.tap_chunks;
        const uint32_t fg = pl.div_wgroups.div(fq), wg = fq - fg * (uint32_t)pl.word_groups;
        const int run = pl.tap_run;
        const int t0 = (int)tchunk * run, wd0 = (int)wg << pl.words_log2;
        const int f0 = (int)fg * PACK_ROWS, ch0 = wd0 * 32;
        const int nch = 32 << pl.words_log2, gt = run << pl.words_log2;          // channels; (word, tap) pairs
        // ---- weights -> one byte each (modes 0, 1: 1 = positive; modes 3, 4: the level's numerator; 0 outside) ----
        // A row is a filter with its channels (mode 1: a channel with its filters), `sub` runs of `run` taps in memory
        // order; its bytes lie in LDS the same way, tap run by tap run.
        const int rows = MODE == 1 ? nch : PACK_ROWS, sub = MODE == 1 ? PACK_ROWS : nch;
        const int pitch = sub * run + 4;
        const int r_real = MODE == 1 ? c - ch0 : k_out - f0, s_real = MODE == 1 ? k_out - f0 : c - ch0;
        const size_t row_stride = (size_t)(MODE == 1 ? k_out : c) * taps;
        const float *base = w + (MODE == 1 ? (size_t)ch0 * row_stride + (size_t)f0 * taps
                                           : (size_t)f0 * row_stride + (size_t)ch0 * taps);
        const int m0 = MODE == 1 ? taps - t0 - run : t0;        // first tap in memory order (may be negative: masked)
        const int len = sub * run;
        // units of 64 consecutive elements of a row, eight in flight per wave
        const int upr = (len + 63) >> 6, units = rows * upr;
        auto stage_bytes = [&](auto whole) {
            for (int u0 = wave; u0 < units; u0 += 4 * 8) {
                float v[8];
                int dst[8];
                bool ok[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int unit = min(u0 + 4 * u, units - 1);
                    const int r = (int)pl.div_units.div_small((uint32_t)unit), i = ((unit - r * upr) << 6) + lane;
                    // (a padded filter group lies past the tensor altogether: masked elements read its first float)
                    const bool real = r < r_real && s_real > 0;
                    const char *src = reinterpret_cast<const char *>(real ? base + (size_t)r * row_stride : w);
                    const int limit = real ? min(s_real, sub) * taps : 0;        // floats of the row that exist here
                    int at = i;
                    if constexpr (whole.value) {                                 // every tap: one run of memory
                        ok[u] = i < limit;
                    } else {
                        const int q = (int)pl.div_tap.div_small((uint32_t)i), m = m0 + i - q * run;
                        at = q * taps + m;
                        ok[u] = i < len && m >= 0 && m < taps && at < limit;
                    }
                    dst[u] = i < len ? r * pitch + i : -1;
                    v[u] = *reinterpret_cast<const float *>(src + (ok[u] ? (uint32_t)at * 4u : 0u));
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (dst[u] >= 0)
                        bytes[dst[u]] = !ok[u] ? 0
                                        : MODE >= 3 ? (uint8_t)(int8_t)(2 * qk_level_index(v[u], levels) - levels)
                                                    : (uint8_t)(v[u] >= 0.0f);
            }
        };
        if (pl.tap_chunks == 1) stage_bytes(std::true_type{});
        else stage_bytes(std::false_type{});
        // byte of (filter f, channel ch, tap tl of the run)
        auto at = [&](int f, int ch, int tl) -> uint32_t {
            return MODE == 1 ? bytes[ch * pitch + f * run + (run - 1 - tl)] : bytes[f * pitch + ch * run + tl];
        };
        if (MODE != 0 && wg == 0 && tchunk == 0 && tid < PACK_ROWS && f0 + tid < k_out)
            alpha[f0 + tid] = MODE >= 3 ? alpha_fill : 1.0f;
        __syncthreads();
        if constexpr (MODE < 3) {
            // lanes are the 32 channels of a word of filters f and f + 1
            for (int q0 = wave; q0 < gt * (PACK_ROWS / 2); q0 += 4 * 4) {
                uint32_t byte[4];
                int slot[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = min(q0 + 4 * u, gt * (PACK_ROWS / 2) - 1);
                    const int pair = q / (PACK_ROWS / 2), f = 2 * (q % (PACK_ROWS / 2)) + (lane >> 5);
                    const int g = (int)pl.div_tap.div_small((uint32_t)pair), tl = pair - g * run;
                    byte[u] = at(f, g * 32 + (lane & 31), tl);
                    slot[u] = pair * PACK_ROWS + f;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const unsigned long long mask = __ballot(byte[u] != 0);
                    if ((lane & 31) == 0) words[slot[u]] = (uint32_t)(lane ? mask >> 32 : mask);
                }
            }
            __syncthreads();
            if (wbits) {
                for (int i = tid; i < gt * PACK_ROWS; i += 256) {     // [filter][tap][word] with the words innermost
                    const int f = (int)pl.div_gt.div_small((uint32_t)i), rem = i - f * gt;
                    const int tl = rem >> pl.words_log2, g = rem & ((1 << pl.words_log2) - 1);
                    if (f0 + f < k_out && t0 + tl < taps && wd0 + g < cw)
                        wbits[((size_t)(f0 + f) * taps + t0 + tl) * cw + wd0 + g] =
                            words[(g * run + tl) * PACK_ROWS + f];
                }
            }
        }
        if (!wmfma) continue;
        // ---- images: every (word, tap) pair is a contiguous run of each --------------------------------------
        const int fb = f0 >> 5, row0 = f0 & 31;
        int8_t *w4 = wmfma + wimg_i8_bytes(k_out, c, taps);
        if constexpr (MODE == 4) {
            const int blocks = taps * cw, recs = (blocks + 1) / 2;
            for (int i = tid; i < gt * PACK_ROWS; i += 256) {
                const int pair = i / PACK_ROWS, f = i % PACK_ROWS;
                const int g = (int)pl.div_tap.div_small((uint32_t)pair), tl = pair - g * run;
                if (t0 + tl >= taps || wd0 + g >= cw) continue;
                uint32_t v[4] = {0, 0, 0, 0};
#pragma unroll
                for (int ch = 0; ch < 32; ++ch)
                    v[ch >> 3] |= Enc<5>::code(at(f, g * 32 + ch, tl)) << (8 * (ch & 3) + (ch & 4));
                const int b = (t0 + tl) * cw + wd0 + g;
                int8_t *rec = w4 + ((size_t)fb * recs + (b >> 1)) * 1024;
                *reinterpret_cast<uint4 *>(rec + (size_t)(row0 + f + 32 * (b & 1)) * 16) = make_uint4(v[0], v[1], v[2], v[3]);
                if (b == blocks - 1 && !(b & 1))    // an odd number of blocks: the last record's other half is zero
                    *reinterpret_cast<uint4 *>(rec + (size_t)(row0 + f + 32) * 16) = make_uint4(0, 0, 0, 0);
            }
            if (blk == 0 && tid < 64)               // the trailing all-zero record
                *reinterpret_cast<uint4 *>(w4 + wimg_f4_bytes(k_out, c, taps) - 1024 + (size_t)tid * 16) = make_uint4(0, 0, 0, 0);
        }
        for (int i = tid; i < gt * PACK_ROWS * 2; i += 256) {
            const int pair = i / (PACK_ROWS * 2), f = i % PACK_ROWS, half = (i / PACK_ROWS) & 1;
            const int g = (int)pl.div_tap.div_small((uint32_t)pair), tl = pair - g * run;
            const int t = t0 + tl, wd = wd0 + g;
            if (t >= taps || wd >= cw) continue;
            uint32_t v[4];
            if constexpr (MODE >= 3) {
                const int ch = g * 32 + half * 16;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[j] = at(f, ch + 4 * j, tl) | at(f, ch + 4 * j + 1, tl) << 8 | at(f, ch + 4 * j + 2, tl) << 16 |
                           at(f, ch + 4 * j + 3, tl) << 24;
            } else {
                const uint32_t bits = words[pair * PACK_ROWS + f] >> (16 * half);
                const int left = f0 + f < k_out ? c - wd * 32 - half * 16 : 0;         // channels from here on
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = left - 4 * j;
                    v[j] = Enc<0>::widen4((bits >> (4 * j)) & 15u) &
                           (r >= 4 ? 0xFFFFFFFFu : r <= 0 ? 0u : (1u << (8 * r)) - 1u);
                }
            }
            const size_t rec = ((size_t)fb * taps + t) * cw + wd;
            *reinterpret_cast<uint4 *>(wmfma + rec * 1024 + (size_t)(row0 + f + 32 * half) * 16) =
                make_uint4(v[0], v[1], v[2], v[3]);
        }
        if (MODE >= 3) {
            if (blk == 0 && tid < 64)           // the trailing all-zero record
                *reinterpret_cast<uint4 *>(w4 - 1024 + (size_t)tid * 16) = make_uint4(0, 0, 0, 0);
            continue;
        }
        const int nblk = taps * cw, nrec = (nblk + 1) / 2;
        uint32_t *wp = reinterpret_cast<uint32_t *>(w4 + wimg_f4_bytes(k_out, c, taps));
        for (int i = tid; i < gt * PACK_ROWS; i += 256) {
            const int pair = i / PACK_ROWS, f = i % PACK_ROWS;
            const int g = (int)pl.div_tap.div_small((uint32_t)pair), tl = pair - g * run;
            const int t = t0 + tl, wd = wd0 + g;
            if (t >= taps || wd >= cw) continue;
            const uint32_t bits = words[i];
            const int b = t * cw + wd;
            int8_t *rec = w4 + ((size_t)fb * nrec + (b >> 1)) * 1024;
            *reinterpret_cast<uint4 *>(rec + (size_t)(row0 + f + 32 * (b & 1)) * 16) =
                Enc<1>::widen_word_regs(bits, f0 + f < k_out, c - wd * 32);
            if (b == nblk - 1 && !(b & 1))      // an odd number of blocks: the last record's other half is zero
                *reinterpret_cast<uint4 *>(rec + (size_t)(row0 + f + 32) * 16) = make_uint4(0, 0, 0, 0);
            wp[((size_t)fb * nblk + b) * 32 + row0 + f] = bits;      // scalar-path image
        }
        if (blk == 0 && tid < 128) {            // the trailing all-zero record of each image
            int8_t *z = tid < 64 ? w4 - 1024 : w4 + wimg_f4_bytes(k_out, c, taps) - 1024;
            *reinterpret_cast<uint4 *>(z + (size_t)(tid & 63) * 16) = make_uint4(0, 0, 0, 0);
        }
    }
}

xnor_status launch_pack_weights(const float *w, uint32_t *wbits, float *alpha, void *wmfma,
                                int k_out, int c, int taps, hipStream_t stream, int mode, int aux, float alpha_fill)
{
    const int cw = (c + 31) / 32;
    PackPlan pl;
    pl.tap_chunks = (taps + PACK_PAIRS - 1) / PACK_PAIRS;
    pl.tap_run = (taps + pl.tap_chunks - 1) / pl.tap_chunks;
    pl.tap_chunks = (taps + pl.tap_run - 1) / pl.tap_run;
    // few taps: several words per workgroup, so that its runs of memory stay long (1x1 filters: 2 KiB per filter)
    pl.words_log2 = 0;
    while ((2 << pl.words_log2) * pl.tap_run <= PACK_PAIRS && (1 << pl.words_log2) < cw) ++pl.words_log2;
    pl.word_groups = (cw + (1 << pl.words_log2) - 1) >> pl.words_log2;
    // the images hold whole blocks of 32 filters, the words only the filters that exist
    const long long fgroups = wmfma ? ((long long)k_out + 31) / 32 * (32 / PACK_ROWS)
                                    : ((long long)k_out + PACK_ROWS - 1) / PACK_ROWS;
    const long long image = fgroups * pl.word_groups * pl.tap_chunks;
    const long long groups = image + (mode == 0 ? k_out : 0);
    if (groups > 0xffffffffLL) return XNOR_ERR_UNSUPPORTED;
    pl.image_groups = (uint32_t)image;
    pl.groups = (uint32_t)groups;
    pl.div_tap = FastDiv::make((uint32_t)pl.tap_run);
    pl.div_gt = FastDiv::make((uint32_t)(pl.tap_run << pl.words_log2));
    pl.div_units = FastDiv::make((uint32_t)(((mode == 1 ? PACK_ROWS : 32 << pl.words_log2) * pl.tap_run + 63) / 64));
    pl.div_chunks = FastDiv::make((uint32_t)pl.tap_chunks);
    pl.div_wgroups = FastDiv::make((uint32_t)pl.word_groups);
    const dim3 grid((unsigned)(groups < (1 << 22) ? groups : (1 << 22))), block(256);      // (larger ones in turns)
#define XNOR_PACK(M) pack_weights_kernel<M><<<grid, block, 0, stream>>>(w, wbits, alpha, (int8_t *)wmfma, k_out, c, taps, cw, (1 << aux) - 1, alpha_fill, pl)
    if (mode == 1) XNOR_PACK(1);
    else if (mode == 3) XNOR_PACK(3);
    else if (mode == 4) XNOR_PACK(4);
    else XNOR_PACK(0);
#undef XNOR_PACK
    return hip_status(hipGetLastError());
}

}  // namespace xnor
