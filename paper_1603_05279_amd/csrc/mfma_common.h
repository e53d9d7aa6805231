// Operand encodings and the LDS plan shared by the matrix-core convolution kernels.
#pragma once
#include "xnor_internal.h"
#include <type_traits>

namespace xnor {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Max-pooling applied in the convolution's epilogue (block order BinConv -> Pool, sec. 3.2).  A pixel tile is
// then a group of `pr` pooled rows of one image: the (pr-1)*sh + ph convolution rows under them, all
// columns, as one run of consecutive flattened output pixels (neighbouring groups overlap by ph - sh rows,
// which are computed twice).
struct PoolPlan {
    int ph, pw, sh, sw;   // window, stride (no padding)
    int hpo, wpo;         // pooled extent
    int pr;               // pooled rows per tile
    int groups;           // tiles per image = ceil(hpo / pr)
    int relu;             // max(., 0) before pooling (the optional ReLU after BinConv)
    FastDiv div_groups, div_wpo;
};

struct MfmaPlan {
    int cc_words;     // channel words per chunk (divides cw; packed words and digits: the last chunk may lack one word, staged as zeros)
    int ps;           // bytes per pixel in LDS (an odd multiple of 16: conflict-free 16-byte reads)
    int max_rows;     // padded input rows a pixel tile can touch
    int region_bytes; // max_rows * row_pitch
    int row_pitch;    // LDS bytes per padded input row (>= wp * ps)
    int nsteps;       // K-steps per chunk
    int tap_jump;     // weight records (packed words: words) skipped when a chunk moves to the next tap
    int ptiles;       // pixel tiles of the launch (the grid is padded beyond it)
    int lut_offset;   // LDS byte offset of the sign-byte widening table
    int ftiles;       // filter tiles of the launch
    int wmajor;       // 1: 1-D grid that keeps the pixel tiles of a filter tile on one XCD
    int vec;          // > 0: channel words per load of the direct staging loop (1 to 4); 0: the general loop
    int quads;        // loads per pixel: cc_words / vec, rounded up
    int dilated;      // direct staging: the input is dilated
    SmallDiv sd_dil_h, sd_dil_w;
    SmallDiv sd_quads, sd_wp, sd_hp, sd_wo, sd_ho;   // direct staging: item, padded and output coordinates of a tile
    int stream_out;   // 1: float results are stored with the non-temporal hint (they exceed a quarter of the last-level cache)
    FastDiv div_wp, div_hp, div_ccw;
    PoolPlan pool;    // used by the pooled-epilogue instantiations only
};

// Direct staging: an item of the staging loop is `vec` channel words of one pixel, read by one load and widened together.
// Coordinates are divided down from the tile's first image with 24-bit multiplies, memory is read through a bounds-checked
// buffer that starts at that image (positions outside an image get an offset beyond it and come back as zero): no 64-bit
// arithmetic, no branch per item.  Needs one chunk that holds every channel word (packed words: or chunks, one after the other;
// 17 images of 384x54x54, 5x5 -> 32, two chunks: 34.9 us with the general loop, 30.8 with this one), and a tile whose images' pixels, packed words and
// padded pixels fit the ranges of those divisions and offsets; anything else takes the general loop.
inline void set_direct_staging(MfmaPlan *pl, const ConvGeom &g, int fmt, int run)
{
    pl->vec = pl->quads = 0;
    if (fmt > 1 || (fmt != 1 && pl->cc_words != g.cw)) return;
    // Odd counts in one chunk: four words too (a load is aligned to a word, not to its size), the last load of a pixel moved back
    // onto the last four, so that some words are loaded and written twice, with the same value.  One word per item
    // repeats the coordinates for each: 16 images of 352x28x28 -> 128 1x1 7.8 -> 6.7 us, 3x3 11.3 -> 9.7, 5x5 17.7 -> 15.0.
    // (chunks of an odd count: the last one may lack a word, single words)
    const bool odd = pl->cc_words == g.cw && g.cw % 2;
    const int vec = odd && g.cw % 3 == 0                     ? 3
                    : odd                                    ? (g.cw > 4 ? 4 : 1)
                    : pl->cc_words % 4 == 0 && g.cw % 4 == 0 ? 4
                    : pl->cc_words % 2 == 0 && g.cw % 2 == 0 ? 2
                                                             : 1;
    const int quads = (pl->cc_words + vec - 1) / vec;
    const long long howo = (long long)g.ho * g.wo, hw = (long long)g.h * g.w;
    const long long images = run / howo + 2;                        // that a tile can touch
    const long long px = (long long)pl->max_rows * g.wp;
    if (images * hw >= (1 << 24) || images * hw * g.cw * 4 >= 0x7fffffffLL || g.cw >= (1 << 22) ||
        px * quads >= (1 << 24) || pl->row_pitch >= (1 << 23) || howo + run >= (1 << 24))
        return;
    pl->dilated = g.dil_h != 1 || g.dil_w != 1;
    if (!SmallDiv::make((uint32_t)g.dil_h, (uint64_t)g.h, &pl->sd_dil_h) || !SmallDiv::make((uint32_t)g.dil_w, (uint64_t)g.w, &pl->sd_dil_w) ||
        !SmallDiv::make((uint32_t)quads, (uint64_t)(px * quads), &pl->sd_quads) ||
        !SmallDiv::make((uint32_t)g.wp, (uint64_t)px, &pl->sd_wp) ||
        !SmallDiv::make((uint32_t)g.hp, (uint64_t)g.hp + pl->max_rows, &pl->sd_hp) ||
        !SmallDiv::make((uint32_t)g.wo, (uint64_t)(howo + run), &pl->sd_wo) ||
        !SmallDiv::make((uint32_t)g.ho, (uint64_t)(howo + run) / g.wo, &pl->sd_ho))
        return;
    pl->vec = vec;
    pl->quads = quads;
}

// Most padded input rows touched by any run of `run` consecutive (flattened) output pixels that
// starts at a multiple of `step`.  The row span only depends on the start modulo the pixels of one
// image, so one period of starts is enough (the host pays a few dozen iterations per launch).
inline int worst_region_rows(const ConvGeom &g, int run, int step)
{
    const long long howo = (long long)g.ho * g.wo;
    // (the validated geometry keeps m_total within 31 bits: 32-bit divisions; a 27 x 27 layer's 243 starts 3.5 -> 2.2 us of
    // host time against 64-bit ones)
    uint32_t a = (uint32_t)step, b = (uint32_t)howo;
    while (b) { const uint32_t t = a % b; a = b; b = t; }       // gcd(step, howo)
    const uint32_t period = (uint32_t)howo / a;
    const uint32_t starts = ((uint32_t)g.m_total + (uint32_t)step - 1) / (uint32_t)step;
    const uint32_t n = starts < period ? starts : period;
    int worst = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const uint32_t m0 = i * (uint32_t)step;
        const uint32_t m1 = (m0 + (uint32_t)run < (uint32_t)g.m_total ? m0 + (uint32_t)run : (uint32_t)g.m_total) - 1;
        const int ia = (int)(m0 / (uint32_t)howo), ib = (int)(m1 / (uint32_t)howo);
        const int oa = (int)((m0 - (uint32_t)ia * (uint32_t)howo) / (uint32_t)g.wo);
        const int ob = (int)((m1 - (uint32_t)ib * (uint32_t)howo) / (uint32_t)g.wo);
        const int rows = (ib * g.hp + ob * g.sh + g.kh - 1) - (ia * g.hp + oa * g.sh) + 1;
        if (rows > worst) worst = rows;
    }
    return worst;
}

template <int FMT> struct Enc;

template <> struct Enc<0> {                    // int8
    static constexpr int BPS = 1;              // channel words per K-step (= per weight record)
    static constexpr int NX = 1;               // matrix instructions per K-step and result block
    static constexpr bool HALF_SPLIT = true;   // a lane's half-wave picks 16 of a word's 32 bytes
    static constexpr int BPB = 32;             // LDS bytes per pixel per channel word
    typedef v16i acc_t;
    static __device__ __forceinline__ acc_t mfma(v4i w, v4i x, acc_t c) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int to_int(acc_t a, int v) { return a[v]; }
    static __device__ __forceinline__ float to_float(acc_t a, int v) { return (float)a[v]; }
    // 4 sign bits -> 4 int8: bit 1 -> 0x01, bit 0 -> 0xFF
    static __device__ __forceinline__ uint32_t widen4(uint32_t nibble) {
        const uint32_t t = __umul24(nibble, 0x00204081u) & 0x01010101u;     // bit i -> byte i
        return __builtin_amdgcn_perm(0x000001FFu, 0x000001FFu, t);           // byte = {0xFF, 0x01}[t]
    }
    // One channel word -> 32 bytes at dst, channels >= nch 0, through a table in LDS: entry b (8 bytes) = the 8 operand bytes of sign byte b,
    // entries 256..511 are zero (selected for positions outside the image).  Three instructions
    // per sign byte instead of a dozen: the widening is instruction-issue bound.
    static constexpr int LUT_BYTES = 512 * 8;
    static __device__ __forceinline__ void build_lut(uint8_t *lut, int tid, int nthreads) {
        uint2 *t = reinterpret_cast<uint2 *>(lut);
        for (int b = tid; b < 512; b += nthreads)
            t[b] = b < 256 ? make_uint2(widen4(b & 15u), widen4((uint32_t)b >> 4)) : make_uint2(0, 0);
    }
    static __device__ __forceinline__ void widen_word_lut(uint8_t *dst, const uint8_t *lut, uint32_t bits, bool ok,
                                                          int nch) {
        const uint8_t *base = lut + (ok ? 0 : 256 * 8);
        const uint2 a = *reinterpret_cast<const uint2 *>(base + (bits & 255u) * 8);
        const uint2 b = *reinterpret_cast<const uint2 *>(base + ((bits >> 8) & 255u) * 8);
        const uint2 c = *reinterpret_cast<const uint2 *>(base + ((bits >> 16) & 255u) * 8);
        const uint2 d = *reinterpret_cast<const uint2 *>(base + (bits >> 24) * 8);
        uint4 lo = make_uint4(a.x, a.y, b.x, b.y), hi = make_uint4(c.x, c.y, d.x, d.y);
        if (nch < 32) {
            uint32_t *p = reinterpret_cast<uint32_t *>(&lo);
            uint32_t *q = reinterpret_cast<uint32_t *>(&hi);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int r0 = nch - 4 * w, r1 = nch - 16 - 4 * w;
                p[w] &= r0 >= 4 ? 0xFFFFFFFFu : (r0 <= 0 ? 0u : (1u << (8 * r0)) - 1u);
                q[w] &= r1 >= 4 ? 0xFFFFFFFFu : (r1 <= 0 ? 0u : (1u << (8 * r1)) - 1u);
            }
        }
        *reinterpret_cast<uint4 *>(dst) = lo;
        *reinterpret_cast<uint4 *>(dst + 16) = hi;
    }
};

template <> struct Enc<1> {                    // 4-bit float E2M1
    static constexpr int BPS = 2;
    static constexpr int NX = 1;
    static constexpr bool HALF_SPLIT = false;  // a lane's half-wave picks one word of the step's pair
    static constexpr int BPB = 16;
    typedef v16f acc_t;
    static __device__ __forceinline__ acc_t mfma(v4i w, v4i x, acc_t c) {
        // 4-bit operands occupy the low four dwords; the rest is left undefined (never read)
        const v8i w8 = __builtin_shufflevector(w, w, 0, 1, 2, 3, -1, -1, -1, -1);
        const v8i x8 = __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1);
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w8, x8, c, 4, 4, 0, 127, 0, 127);
    }
    static __device__ __forceinline__ int to_int(acc_t a, int v) { return (int)a[v]; }
    static __device__ __forceinline__ float to_float(acc_t a, int v) { return a[v]; }   // an exact integer already
    // 8 sign bits -> 8 nibbles (bit 1 -> 0x2, +1.0; bit 0 -> 0xA, -1.0) with one byte permute: an output byte holds two channels, i.e. one of four values
    // (0xAA, 0xA2, 0x2A, 0x22 for the bit pairs 00, 01, 10, 11), and v_perm_b32 picks four bytes out of a 32-bit
    // table by four selector bytes.  The selectors are the byte's four bit pairs spread to byte positions by two
    // shift-ors and a mask: four vector instructions per output dword, no table in LDS (whose reads would hit
    // random banks).  `byte` must be clean above bit 7.
    static __device__ __forceinline__ uint32_t widen8_perm(uint32_t byte, uint32_t tbl = 0x222AA2AAu) {
        uint32_t t = (byte << 6) | byte;
        t = (t << 12) | t;
        return __builtin_amdgcn_perm(0u, tbl, t & 0x03030303u);
    }
    static constexpr int LUT_BYTES = 0;
    static __device__ __forceinline__ void build_lut(uint8_t *, int, int) {}
    static __device__ __forceinline__ uint4 widen_word_regs(uint32_t bits, bool ok, int nch) {
        // positions outside the image pick from an all-zero table (code 0x0 = 0.0)
        const uint32_t tbl = ok ? 0x222AA2AAu : 0u;
        uint4 v;
        v.x = widen8_perm(bits & 255u, tbl);
        v.y = widen8_perm((bits >> 8) & 255u, tbl);
        v.z = widen8_perm((bits >> 16) & 255u, tbl);
        v.w = widen8_perm(bits >> 24, tbl);
        if (nch < 32) {
            uint32_t *d = reinterpret_cast<uint32_t *>(&v);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r0 = nch - 8 * q;
                d[q] &= r0 >= 8 ? 0xFFFFFFFFu : (r0 <= 0 ? 0u : (1u << (4 * r0)) - 1u);
            }
        }
        return v;
    }
    // Operand order of the convolution: dword q of a word's 16 bytes holds in nibble j channel 4j + 3 - q, so that a dword
    // is one shift and one and-or of the packed word (7 vector instructions per word; canonical nibble order takes 17).  A
    // sign bit of 1 becomes 0xA (-1), of 0 becomes 0x2 (+1): inverted in both operands alike, which leaves their products
    // what they are.  `code` has the sign positions that exist (0x88888888, per lane 0 for a block that must not count).
    static __device__ __forceinline__ v4i widen_bits(uint32_t bits, uint32_t code, uint32_t one) {    // one = code >> 2
        return v4i{(int)((bits & code) | one), (int)(((bits << 1) & code) | one), (int)(((bits << 2) & code) | one),
                   (int)(((bits << 3) & code) | one)};
    }
    static __device__ __forceinline__ void widen_word_lut(uint8_t *dst, const uint8_t *, uint32_t bits, bool ok,
                                                          int nch) {
        // positions outside the image: code 0x0 = 0.0
        v4i v = widen_bits(bits, ok ? 0x88888888u : 0u, ok ? 0x22222222u : 0u);
        if (nch < 32) {                                       // channels past the last one: 0.0 too
            const uint32_t real = (1u << nch) - 1u;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] &= (int)((((real << q) & 0x88888888u) >> 3) * 15u);
        }
        *reinterpret_cast<v4i *>(dst) = v;
    }
};


constexpr int ring_lcm(int a, int b)
{
    int m = a;
    while (m % b) m += a;
    return m;
}

// Binary-Weight-Network operands (sec. 3.1: real inputs, +-1 weights).  A word is 32 channels of a pixel, staged as five
// digits of 6-bit floats (E2M3) with one power-of-two scale 2^e, 2^e <= max |x| < 2^(e+1) over the word:
//     x = 2^e * (d0 + d1 / 32 + d2 / 32^2 + d3 / 32^3 + d4 / 32^4),   |d| <= 2 in steps of 1/8 (all of them E2M3 values),
// each digit the nearest to what the digits before it left (those remainders are exact).  The last digit's step is the unit in
// the last place of the word's largest input: that one is represented exactly, the others to half of that unit, which
// is what a float sum that the largest one enters can hold of them (every filter adds all 32, weights are never 0).
// Where |x| >= 2^127 the first digit is at most 1.875 and the next ones reach 4 in steps of 1/4: inputs from 1.9375 * 2^127 on
// are held to a unit in the last place.
// The matrix instruction multiplies E2M3 by the +-1 weights (E2M1, widened from packed bits as in the binary
// convolution), applies the scales (activations: e, weights: the digit's 32^-k) and accumulates in float; 5 instructions of the
// 4- and 6-bit rate per 64 channels take the place of 12 bfloat16 ones (three parts).
// A word with an infinite or NaN input has the scale NaN: every result that it enters is NaN.  e is at least -106
// (scales of all digits stay normal floats): inputs below keep an absolute error of 2^-130.
template <> struct Enc<2> : Enc<1> {
    static constexpr int DIGITS = 5;
    static constexpr int BPB = 128;            // five 24-byte operands, the scale, 4 bytes of padding
    static constexpr int SCALE_DWORD = 30;
    static constexpr int MIN_FIELD = 21;       // biased exponent of the smallest scale
    typedef unsigned v6u __attribute__((ext_vector_type(6)));
    typedef int v32i __attribute__((ext_vector_type(32)));
    typedef float v16 __attribute__((ext_vector_type(16)));
    typedef float v32 __attribute__((ext_vector_type(32)));
    // K position of channel ch in the 4-bit operands (widen_bits): 8 * (3 - ch % 4) + ch / 4.  The conversion of two
    // 16-vectors puts lo[i] at position 2i and hi[i] at 2i + 1.
    static constexpr int channel_at(int pos) { return 4 * (pos % 8) + 3 - pos / 8; }
    // x: the word's channels in order.  out: the 32 dwords of the staged word.
    static __device__ __forceinline__ void digits(const float (&x)[32], uint32_t (&out)[32])
    {
        uint32_t m = 0;
#pragma unroll
        for (int c = 0; c < 32; ++c) m = max(m, __builtin_bit_cast(uint32_t, x[c]) & 0x7fffffffu);
        const uint32_t field = max(m >> 23, (uint32_t)MIN_FIELD);
        v16 lo, hi;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            lo[i] = x[channel_at(2 * i)];
            hi[i] = x[channel_at(2 * i + 1)];
        }
#pragma unroll
        for (int k = 0; k < DIGITS; ++k) {
            const float scale = __builtin_bit_cast(float, (field - 5u * k) << 23);
            v16 l = lo, h = hi;
            if (k == 0 && field == 254u) {       // the top binade: a first digit of 2 would stand for 2^128, which is no float
                const float top = 1.875f * 0x1p127f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    l[i] = __builtin_fminf(__builtin_fmaxf(l[i], -top), top);
                    h[i] = __builtin_fminf(__builtin_fmaxf(h[i], -top), top);
                }
            }
            const v6u d = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(l, h, scale);
#pragma unroll
            for (int i = 0; i < 6; ++i) out[6 * k + i] = d[i];
            if (k + 1 < DIGITS) {
                const v32 back = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(d, scale);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    lo[i] -= back[2 * i];
                    hi[i] -= back[2 * i + 1];
                }
            }
        }
        out[SCALE_DWORD] = field;
        out[31] = 0;
    }
    template <int K> static __device__ __forceinline__ acc_t mfma_digit(v4i w, const v32i &x, acc_t c)
    {
        const v8i w8 = __builtin_shufflevector(w, w, 0, 1, 2, 3, -1, -1, -1, -1);
        const v8i x8 = __builtin_shufflevector(x, x, 6 * K, 6 * K + 1, 6 * K + 2, 6 * K + 3, 6 * K + 4, 6 * K + 5, -1, -1);
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w8, x8, c, 4, 2, 0, 127 - 5 * K, 0, x[SCALE_DWORD]);
    }
};

// Binary-Weight-Network operands without conversion, where the split writes parts (bwn_in_digits) and the K loop is so short (few taps, few
// workgroups) that making the digits above while staging would take longer than their matrix instructions save.  The real activations arrive
// pre-split into three bfloat16 parts (hi + mid + lo == the float exactly), 16 channels x one part
// = one 32-byte "word" per pixel; the weights are +-1.0 (0 past the last channel or filter) in
// bfloat16, one record per 16-channel group that multiplies all three parts (the record is fetched
// once per K-step and feeds three matrix instructions per result block).  Products are exact,
// accumulation is float: the result is the float sum of exact terms.  Layout-wise a word is like the
// int8 encoding's (32 bytes per pixel and word, the half-wave picks its 16 bytes), with nothing to widen.
template <> struct Enc<4> {
    static constexpr int BPS = 3;       // a K-step = one 16-channel group = the three parts' words, one weight record
    static constexpr int NX = 3;        // matrix instructions per step and result block (one per part)
    static constexpr bool HALF_SPLIT = true;
    static constexpr int BPB = 32;
    typedef v16f acc_t;
    typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
    static __device__ __forceinline__ acc_t mfma(v4i w, v4i x, acc_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, w), __builtin_bit_cast(v8bf, x), c, 0, 0,
                                                       0);
    }
    static __device__ __forceinline__ int to_int(acc_t a, int v) { return (int)a[v]; }
    static __device__ __forceinline__ float to_float(acc_t a, int v) { return a[v]; }
    static constexpr int LUT_BYTES = 0;
    static __device__ __forceinline__ void build_lut(uint8_t *, int, int) {}
};

// The same parts, made from digits (Enc<2>) while they are staged: for filters so tall that one channel word's digits of the rows under a
// tile do not fit the LDS and a part of 16 channels does.
template <> struct Enc<6> : Enc<4> {
    // word: the 32 dwords of 32 channels' digits; half: which 16 of them; out: their hi, mid and lo parts, 16 bfloat16 numbers each
    static __device__ __forceinline__ void parts_of_digits(const v4u (&word)[8], int half, v4u (&out)[6])
    {
        typedef Enc<2> D;
        const uint32_t field = word[D::SCALE_DWORD / 4][D::SCALE_DWORD % 4];
        float x[32];
#pragma unroll
        for (int k = D::DIGITS - 1; k >= 0; --k) {
            D::v6u d;
#pragma unroll
            for (int i = 0; i < 6; ++i) d[i] = word[(6 * k + i) / 4][(6 * k + i) % 4];
            const D::v32 back = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(d, __builtin_bit_cast(float, (field - 5u * k) << 23));
#pragma unroll
            for (int i = 0; i < 32; ++i) {        // (smallest first: every sum is a float)
                const int ch = D::channel_at(i);
                x[ch] = k == D::DIGITS - 1 ? back[i] : x[ch] + back[i];
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float a = half ? x[16 + 2 * i] : x[2 * i], b = half ? x[17 + 2 * i] : x[2 * i + 1];
            if (field == 255u) a = b = __builtin_nanf("");       // a word with an infinite or NaN input
#pragma unroll
            for (int part = 0; part < 3; ++part) {
                const uint32_t ha = bf16_rne(a), hb = bf16_rne(b);
                out[2 * part + i / 4][i % 4] = ha | (hb << 16);
                a -= bf16_value(ha);
                b -= bf16_value(hb);
            }
        }
    }
};

// k-bit quantised operands (sec. 3.2, "k-bit Quantization"): activations and weights arrive as the odd-integer
// numerators 2u - L of their levels in int8 (32 channels = one 32-byte word per pixel, 0 past the last
// channel), so the int8 matrix instruction accumulates the exact integer sum of products; nothing to widen.
template <> struct Enc<3> : Enc<0> {
    static constexpr int LUT_BYTES = 0;
    static __device__ __forceinline__ void build_lut(uint8_t *, int, int) {}
};

// k-bit operands of at most two bits each: the numerators +-1 and +-3 are 4-bit floats (E2M1 0x2, 0x5 and their negatives), so the
// contraction runs at twice the int8 rate on operands of half the size; its float sums are exact while they stay below 2^24.
// Dword q of a word holds channel 8q + i in nibble 2i and channel 8q + 4 + i in nibble 2i + 1.
template <> struct Enc<5> : Enc<1> {
    // int8 numerators -> codes: (byte >> 1) & 3 is 0, 1, 2, 3 for 1, 3, -3, -1 (channels past the last one are 0 there, and
    // 0 in the weights)
    static constexpr uint32_t CODES = 0x0A0D0502u;
    static __device__ __forceinline__ v4i narrow(v4u lo, v4u hi) {
        v4i r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t a = q < 2 ? lo[2 * q] : hi[2 * q - 4], b = q < 2 ? lo[2 * q + 1] : hi[2 * q - 3];
            r[q] = (int)(__builtin_amdgcn_perm(0u, CODES, (a >> 1) & 0x03030303u) |
                         __builtin_amdgcn_perm(0u, CODES, (b >> 1) & 0x03030303u) << 4);
        }
        return r;
    }
    static __device__ __forceinline__ uint32_t code(uint32_t byte) { return byte ? (CODES >> (4 * (byte & 6u))) & 15u : 0u; }
};

// Steps the offset table is padded by beyond the last K-step (copies of the last entry): operand
// prefetches run ahead of the loop's end by at most one turn plus the activation depth.
constexpr int KLOOP_TABLE_PAD = 20;

// Weight record stream of a chunk that holds every channel word: the records of a filter block are
// consecutive, so each block gets its own buffer resource covering exactly nsteps records and the
// lane's offset advances by 1 KiB per step.  Prefetches past the end (never multiplied) fall outside
// the resource and are answered with zeros by the buffer bounds check instead of touching memory;
// the check covers the vector offset only, which is why the step lives there and not in the scalar
// offset.  No other bookkeeping in the loop.
// AUX: cache policy of the loads (2 = non-temporal hint).
template <int FW, int AUX = 0> struct WStreamLinear {
    typedef v4i word_t;
    static constexpr bool WIDEN = false;
    __amdgpu_buffer_rsrc_t rsrc[FW];
    int voff;
    __device__ __forceinline__ WStreamLinear(const v4i *wimg, const int (&wrec0)[FW], int rec_start, int nsteps,
                                             int wlane)
        : voff(wlane)
    {
#pragma unroll
        for (int i = 0; i < FW; ++i)
            rsrc[i] = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<v4i *>(wimg + (size_t)(wrec0[i] + rec_start) * 64), 0, nsteps * 1024, 0x00020000);
    }
    __device__ __forceinline__ void load(v4i (&dst)[FW])
    {
#pragma unroll
        for (int i = 0; i < FW; ++i) {
            const v4u r = __builtin_amdgcn_raw_buffer_load_b128(rsrc[i], voff, 0, AUX);
            dst[i] = v4i{(int)r[0], (int)r[1], (int)r[2], (int)r[3]};
        }
        voff += 1024;
    }
};

// Weight record stream of a chunk that holds part of the channel words: +1 record per step and
// +tap_jump more when the chunk moves to the next tap; steps past the end read the all-zero record.
// Branch-free scalar bookkeeping, so the loop body stays one basic block.
template <int FW> struct WStreamChunked {
    typedef v4i word_t;
    static constexpr bool WIDEN = false;
    __amdgpu_buffer_rsrc_t rsrc;
    int wrec0[FW];
    int wlane, zero_rec, w_rec, w_cnt, w_left, steps_per_tap, tap_jump;
    __device__ __forceinline__ WStreamChunked(__amdgpu_buffer_rsrc_t rsrc_, const int (&wrec0_)[FW], int zero_rec_,
                                              int rec_start, int nsteps, int steps_per_tap_, int tap_jump_,
                                              int wlane_)
        : rsrc(rsrc_), wlane(wlane_), zero_rec(zero_rec_), w_rec(rec_start), w_cnt(0), w_left(nsteps),
          steps_per_tap(steps_per_tap_), tap_jump(tap_jump_)
    {
#pragma unroll
        for (int i = 0; i < FW; ++i) wrec0[i] = wrec0_[i];
    }
    __device__ __forceinline__ void load(v4i (&dst)[FW])
    {
        const int live = w_left > 0 ? 1 : 0;
#pragma unroll
        for (int i = 0; i < FW; ++i) {
            const int rec = live ? wrec0[i] + w_rec : zero_rec;
            const v4u r = __builtin_amdgcn_raw_buffer_load_b128(rsrc, wlane, rec * 1024, 0);
            dst[i] = v4i{(int)r[0], (int)r[1], (int)r[2], (int)r[3]};
        }
        w_left -= live;
        w_cnt += live;
        const int wrap = w_cnt == steps_per_tap ? 1 : 0;
        w_cnt = wrap ? 0 : w_cnt;
        w_rec += live + (wrap ? tap_jump : 0);
    }
};

// Weight stream of the 4-bit operands: the packed words themselves, [filter block][(tap, channel word)][32 filters], two
// (tap, word) blocks = 256 bytes per K-step and filter block, one word per lane, widened in registers while the matrix
// pipes work on the step before (a matrix instruction leaves its wave seven issue slots).  Each filter block has a
// resource of its own that ends with its words: reads beyond are answered with zeros, as above only while the step lies in the
// vector offset.  When the block count is odd the second half-wave of the last step holds no block: its code is 0 (operand 0.0).
// Steps are consecutive (LINEAR) or, where a chunk holds part of the channel words, run on within a tap and skip
// tap_jump words to the next one (uniform bookkeeping, one vector addition per step; steps past the end read the block's
// first words, which nothing multiplies).  Where a chunk holds one of several channel words a step takes it of two taps, whose blocks
// lie half_blk apart.  There too the second half-wave of a filter's very last step may lie beyond its
// words: a last chunk that lacks a word, an odd block count in one chunk.
template <int FW, bool LINEAR, int AUX = 0> struct WStreamBits {
    typedef uint32_t word_t;
    static constexpr bool WIDEN = true;
    __amdgpu_buffer_rsrc_t rsrc[FW];
    int voff, w_blk, w_cnt, w_left, steps_per_tap, tap_jump;
    uint32_t last_code;          // code of the last step
    __device__ __forceinline__ WStreamBits() = default;
    __device__ __forceinline__ WStreamBits(const uint32_t *words, const int (&fblk)[FW], int nblk, int first,
                                           int nsteps, bool odd_last, int lane, int steps_per_tap_, int tap_jump_, int half_blk = 1)
        : voff((lane & 31) * 4 + (lane >> 5) * half_blk * 128 + (LINEAR ? first * 128 : 0)), w_blk(first), w_cnt(0), w_left(nsteps),
          steps_per_tap(steps_per_tap_), tap_jump(tap_jump_), last_code(odd_last && lane >= 32 ? 0u : 0x88888888u)
    {
#pragma unroll
        for (int i = 0; i < FW; ++i)
            rsrc[i] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(words) + (size_t)fblk[i] * nblk * 32, 0,
                                                        nblk * 128, 0x00020000);
    }
    __device__ __forceinline__ void load(word_t (&dst)[FW])
    {
#pragma unroll
        for (int i = 0; i < FW; ++i)
            dst[i] = __builtin_amdgcn_raw_buffer_load_b32(rsrc[i], LINEAR ? voff : voff + w_blk * 128, 0, AUX);
        if constexpr (LINEAR) {
            voff += 256;
        } else {
            const int live = w_left > 0 ? 1 : 0;
            w_left -= live;
            w_cnt += live;
            const int wrap = w_cnt == steps_per_tap ? 1 : 0;
            w_cnt = wrap ? 0 : w_cnt;
            w_blk += 2 * live + (wrap ? tap_jump : 0);
            w_blk = w_left > 0 ? w_blk : 0;
        }
    }
};

// Keeps an accumulator where it is at this place of the code: matrix instructions before it stay before it.  ACC: the wave has a
// SIMD to itself and its accumulators lie in the accumulation registers, a pin to vector registers would move all of them there
// and back (pooled epilogue, 160-pixel tiles, 11 images of 128 x 38 x 38, 3 x 3 -> 256: 20.1 us with it, 16.3 without).
template <bool ACC, class A> __device__ __forceinline__ void pin_acc(A &acc)
{
    if constexpr (ACC) asm volatile("" : "+a"(acc));
    else asm volatile("" : "+v"(acc));
}

// One chunk's K loop of a wave: acc[i][j] += W(filter block i, step s) x X(pixel block j, step s)
// for s = 0 .. nsteps-1, weights from the stream `ws` (one of those above), activations from LDS
// through the per-step offset table (padded by KLOOP_TABLE_PAD steps).  The first DW steps' weights are on their way already (w).  Operands are requested DW
// steps (weights: buffer loads with a scalar offset, L2 latency) and DX steps (activations) ahead
// of their use and live in register rings of DW+1 and DX+1 slots; the body is unrolled until both
// rings are back at slot 0.  Packed weight words are widened one step ahead of their use.  A wave issues one
// instruction every four cycles, so everything that is
// not a matrix instruction competes with them for issue slots: the loop carries no address or
// bounds arithmetic beyond PW + 1 vector adds per step.
// The scheduling barriers pin the order written here (next operands requested, then the current
// step's matrix instructions interleaved with those requests), which the compiler otherwise
// regroups into one burst of loads followed by one burst of MFMAs with the latencies exposed.
template <class E, int FW, int PW, int DW, int DX, class WS>
__device__ __forceinline__ void mfma_kloop(typename E::acc_t (&acc)[FW][PW], const uint8_t *lds_x,
                                           const int (&pbase)[PW], const int *xoff_tab, int tab_lane, WS &ws,
                                           typename WS::word_t (&w)[DW + 1][FW], int nsteps)
{
    constexpr int RW = DW + 1, RX = DX + 1;
    constexpr int TURN = ring_lcm(RW, RX);     // sub-steps after which both rings are back at slot 0
    static_assert(RX <= RW && TURN <= 16 && TURN % 2 == 0, "unrolled turn: even, at most 16 sub-steps");
    static_assert(TURN + DX + 2 <= KLOOP_TABLE_PAD, "offset table padding");
    typedef typename WS::word_t word_t;
    const int *tab = xoff_tab + tab_lane;
    auto load_t = [&](int s) -> int { return tab[s * E::BPS]; };
    constexpr int NX = E::NX;                  // words of a step that share its weight record
    auto load_x = [&](v4i (&dst)[PW][NX], int toff) {
#pragma unroll
        for (int j = 0; j < PW; ++j)
#pragma unroll
            for (int q = 0; q < NX; ++q)
                dst[j][q] = *reinterpret_cast<const v4i *>(lds_x + pbase[j] + toff + q * E::BPB);
    };
    auto fma_all = [&](const v4i (&w)[FW], const v4i (&x)[PW][NX]) {
#pragma unroll
        for (int q = 0; q < NX; ++q)
#pragma unroll
            for (int j = 0; j < PW; ++j)
#pragma unroll
                for (int i = 0; i < FW; ++i) acc[i][j] = E::mfma(w[i], x[j][q], acc[i][j]);
    };

    v4i x[RX][PW][NX], wide[2][FW];
    int tq[2];
    // (in registers: an and-or takes no two literals)
    uint32_t full = 0x88888888u, full_one = 0x22222222u;
    if constexpr (WS::WIDEN) asm("" : "+v"(full), "+v"(full_one));
    auto widen = [&](v4i (&dst)[FW], const word_t (&src)[FW], int s, bool tail) {
        if constexpr (WS::WIDEN) {
            // every step but the last counts both half-waves
            const uint32_t code = tail && s == nsteps - 1 ? ws.last_code : full;
            const uint32_t one = tail && s == nsteps - 1 ? ws.last_code >> 2 : full_one;
#pragma unroll
            for (int i = 0; i < FW; ++i) dst[i] = E::widen_bits(src[i], code, one);
        }
    };
#pragma unroll
    for (int u = 0; u < DX; ++u) load_x(x[u], load_t(u));
    tq[0] = load_t(DX);
    widen(wide[0], w[0], 0, true);
    auto substep = [&](int s, int u, bool tail) {
        ws.load(w[(u + DW) % RW]);                      // step s+u+DW
        tq[(u + 1) & 1] = load_t(s + u + DX + 1);
        load_x(x[(u + DX) % RX], tq[u & 1]);            // step s+u+DX, offset read one sub-step ago
        if constexpr (WS::WIDEN) {
            fma_all(wide[u & 1], x[u % RX]);
            widen(wide[(u + 1) & 1], w[(u + 1) % RW], s + u + 1, tail);
        } else {
            fma_all(w[u % RW], x[u % RX]);
        }
        // one LDS read behind each of the first PW*NX+1 MFMAs, then the FW weight loads; widening instructions fill the
        // slots behind all of them
        constexpr int MM = FW * PW * NX, VALU = WS::WIDEN ? 7 * FW : 0;
#pragma unroll
        for (int q = 0; q < MM; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (q < PW * NX + 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            else if (q < PW * NX + 1 + FW) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            if (VALU) __builtin_amdgcn_sched_group_barrier(0x002, (VALU + MM - 1) / MM, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 0;
    for (; s + TURN < nsteps; s += TURN) {              // whole turns but the last: one basic block, no exits
#pragma unroll
        for (int u = 0; u < TURN; ++u) substep(s, u, u == TURN - 1);
    }
    // the last turn.  The accumulators are pinned before every exit test: otherwise the
    // matrix instructions sink below the branches and run in one burst behind all the loads.
#pragma unroll
    for (int u = 0; u < TURN; ++u) {
        if (s + u >= nsteps) break;
        substep(s, u, true);
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int j = 0; j < PW; ++j) pin_acc<(FW * PW > 8)>(acc[i][j]);
    }
}

// The K loop of the digit operands (Enc<2>): a step is 64 channels, five matrix instructions per result block.  One pixel
// block's digits (128 bytes per lane, eight reads) are read while the block before it is multiplied.
template <int FW, int PW, int DW, class WS>
__device__ __forceinline__ void mfma_kloop_digits(Enc<2>::acc_t (&acc)[FW][PW], const uint8_t *lds_x,
                                                  const int (&pbase)[PW], const int *xoff_tab, int tab_lane, WS &ws,
                                                  typename WS::word_t (&w)[DW + 1][FW], int nsteps)
{
    typedef Enc<2> E;
    constexpr int RW = DW + 1;
    static_assert(RW % 2 == 0 && RW + 3 <= KLOOP_TABLE_PAD, "rings");
    // a wave tile of one result block alternates between two sums: a matrix instruction takes twice its rate to its result
    constexpr bool TWO = FW * PW == 1;
    E::acc_t odd;
    if constexpr (TWO) {
#pragma unroll
        for (int v = 0; v < 16; ++v) odd[v] = 0.0f;
    }
    const int *tab = xoff_tab + tab_lane;
    v4i wide[2][FW];
    uint32_t full = 0x88888888u, full_one = 0x22222222u;
    asm("" : "+v"(full), "+v"(full_one));
    auto widen = [&](v4i (&dst)[FW], const typename WS::word_t (&src)[FW], int s, bool tail) {
        const uint32_t code = tail && s == nsteps - 1 ? ws.last_code : full;
        const uint32_t one = tail && s == nsteps - 1 ? ws.last_code >> 2 : full_one;
#pragma unroll
        for (int i = 0; i < FW; ++i) dst[i] = E::widen_bits(src[i], code, one);
    };
    auto load_x = [&](E::v32i &dst, int at) {
        v4i d[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) d[q] = *reinterpret_cast<const v4i *>(lds_x + at + 16 * q);
#pragma unroll
        for (int q = 0; q < 32; ++q) dst[q] = d[q / 4][q % 4];
    };
    E::v32i x[2];
    int off = tab[0], off_next = tab[E::BPS];
    load_x(x[0], pbase[0] + off);
    widen(wide[0], w[0], 0, true);
    auto substep = [&](int s, int u, bool tail) {
        ws.load(w[(u + DW) % RW]);
        const int off_after = tab[(s + u + 2) * E::BPS];
#pragma unroll
        for (int j = 0; j < PW; ++j) {
            const E::v32i &cur = x[(u * PW + j) & 1];
            load_x(x[(u * PW + j + 1) & 1], j + 1 < PW ? pbase[j + 1] + off : pbase[0] + off_next);
            auto digit = [&](auto k) {
                constexpr int K = decltype(k)::value;
#pragma unroll
                for (int i = 0; i < FW; ++i) {
                    E::acc_t &a = TWO && K % 2 ? odd : acc[i][j];
                    a = E::mfma_digit<K>(wide[u & 1][i], cur, a);
                }
            };
            digit(std::integral_constant<int, 0>{});
            digit(std::integral_constant<int, 1>{});
            digit(std::integral_constant<int, 2>{});
            digit(std::integral_constant<int, 3>{});
            digit(std::integral_constant<int, 4>{});
            if (j == PW - 1) widen(wide[(u + 1) & 1], w[(u + 1) % RW], s + u + 1, tail);
            // two reads behind each of the first four matrix instructions, the rest of the slots for the widening
#pragma unroll
            for (int q = 0; q < 5 * FW; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (q < 5) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        off = off_next;
        off_next = off_after;
    };
    int s = 0;
    for (; s + RW < nsteps; s += RW) {
#pragma unroll
        for (int u = 0; u < RW; ++u) substep(s, u, u == RW - 1);
    }
#pragma unroll
    for (int u = 0; u < RW; ++u) {
        if (s + u >= nsteps) break;
        substep(s, u, true);
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int j = 0; j < PW; ++j) pin_acc<(FW * PW > 6)>(acc[i][j]);
    }
    if constexpr (TWO) acc[0][0] += odd;
}

}  // namespace xnor
