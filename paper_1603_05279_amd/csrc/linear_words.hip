// Fully connected layers on the matrix cores (footnote of sec. 1: a convolution whose filter covers the whole input), both operands
// widened from packed words in registers.
#include "mfma_common.h"
#include "linear_route.h"
#include <atomic>

namespace xnor {

// A workgroup makes 32 * FW filters x 32 * PW rows; its KW waves share the words of a row in groups of eight (four K-steps: half-wave h
// takes words 8q + 4h .. + 3, the rows' with one 16-byte load per lane, the filters' with one load per word from the packed image,
// [filter block][word][32 filters]).  The waves' sums, exact integers, meet in LDS.  Nothing is staged: every wave has rows and filters of its
// own, so an operand in LDS would be read once.
// What bounds it: the vector instructions of the widening (7 per word, 31 for the four matrix instructions of a step of the largest tile: 50
// cycles each at a wave's or a SIMD's rate, against 36 for the matrix pipe), then two trips to memory and the launch.  Staging the rows in LDS
// instead (conv_mfma_kernel, 128 x 32 tiles) cost 1.3 us of set-up and 3.6 of widening 147 KB per workgroup ahead of 4.2 us of K loop: back to
// back 256 rows 9216 -> 4096 13.4 -> 9.0 us, 128 rows 13.2 -> 6.5, 64 rows 13.3 -> 4.8, 256 rows 4096 -> 1000 8.5 -> 4.2, 25088 -> 4096 58 -> 18.
// (Four waves per workgroup 11.4 us, sixteen with tiles of 32 x 32 13.3, against 9.1.)
// Groups reach past the last word: the last load of a row is moved back onto its last four words, and what an earlier word of the
// group has counted is taken out of the filters' operand (code 0, 0.0).  Channels past the last one are 0 bits on both sides, +1 each:
// subtracted from the sum.
typedef uint32_t words4 __attribute__((ext_vector_type(4), aligned(4)));      // (16-byte loads of rows that are aligned to words)

struct LinearWordsArgs {
    const uint32_t *xbits, *words;
    const float *Krow, *alpha;
    float *out;
    int32_t *dot_out;
    int n, cw, k_out, fblocks, pad, ptiles, ftiles, wmajor;
};

template <int FW, int PW, int KW>
__global__ __launch_bounds__(64 * KW) void linear_words_kernel(LinearWordsArgs a)
{
    typedef Enc<1> E;
    constexpr int FT = 32 * FW, RT = 32 * PW, PITCH = FT + 4;      // LDS floats per row: 16-byte accesses of neighbouring rows on different banks
    constexpr int D = 2;                                           // groups in flight per wave
    extern __shared__ __attribute__((aligned(16))) float red[];    // [KW][RT][PITCH]
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // filter tiles of 8 XCDs in turn, all row tiles of one on the same XCD, whose L2 then reads its words once
    int ftile, ptile;
    if (a.wmajor) {
        const int slot = blockIdx.x >> 3;
        ftile = slot / a.ptiles * 8 + (blockIdx.x & 7);
        ptile = slot % a.ptiles;
        if (ftile >= a.ftiles) return;
    } else {
        ftile = blockIdx.x / a.ptiles;
        ptile = blockIdx.x % a.ptiles;
    }
    const int f0 = ftile * FT, n0 = ptile * RT;
    const uint32_t *xrow[PW], *wcol[FW];
#pragma unroll
    for (int j = 0; j < PW; ++j) xrow[j] = a.xbits + (size_t)min(n0 + 32 * j + l32, a.n - 1) * a.cw;
#pragma unroll
    for (int i = 0; i < FW; ++i) wcol[i] = a.words + (size_t)min(f0 / 32 + i, a.fblocks - 1) * a.cw * 32 + l32;
    const int groups = (a.cw + 7) >> 3;
    words4 x[D][PW];
    uint32_t w[D][FW][4];
    auto load = [&](int u, int q) {
        const int w0 = min(8 * q + 4 * half, a.cw - 4);
#pragma unroll
        for (int j = 0; j < PW; ++j) x[u][j] = *reinterpret_cast<const words4 *>(xrow[j] + w0);
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int s = 0; s < 4; ++s) w[u][i][s] = wcol[i][(size_t)(w0 + s) * 32];
    };
    E::acc_t acc[FW][PW];
#pragma unroll
    for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int j = 0; j < PW; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    uint32_t full = 0x88888888u, full_one = 0x22222222u;
    asm("" : "+v"(full), "+v"(full_one));          // (in registers: an and-or takes no two literals)
    auto multiply = [&](int u, int q) {
        const int first = 8 * q + 4 * half - min(8 * q + 4 * half, a.cw - 4);     // words of the load that an earlier one counted
        const bool tail = 8 * q + 8 > a.cw;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint32_t code = tail && s < first ? 0u : full, one = tail && s < first ? 0u : full_one;
            v4i wx[PW], ww[FW];
#pragma unroll
            for (int i = 0; i < FW; ++i) ww[i] = E::widen_bits(w[u][i][s], code, one);
#pragma unroll
            for (int j = 0; j < PW; ++j) wx[j] = E::widen_bits(x[u][j][s], full, full_one);
#pragma unroll
            for (int j = 0; j < PW; ++j)
#pragma unroll
                for (int i = 0; i < FW; ++i) acc[i][j] = E::mfma(ww[i], wx[j], acc[i][j]);
        }
    };
#pragma unroll
    for (int u = 0; u < D; ++u)
        if (wave + u * KW < groups) load(u, wave + u * KW);
    for (int q = wave; q < groups; q += D * KW) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (q + u * KW >= groups) break;
            multiply(u, q + u * KW);
            if (q + (u + D) * KW < groups) load(u, q + (u + D) * KW);
        }
    }
    // the waves' sums; each thread then adds those of four neighbouring filters of a row
    constexpr int QUADS = FT / 4, OUTS = RT * QUADS, PER = (OUTS + 64 * KW - 1) / (64 * KW);
    float Kr[PER], al[PER][4];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int idx = min(tid + p * 64 * KW, OUTS - 1), row = n0 + idx / QUADS, f = f0 + idx % QUADS * 4;
        Kr[p] = a.Krow[min(row, a.n - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) al[p][q] = a.alpha[min(f + q, a.k_out - 1)];
    }
#pragma unroll
    for (int j = 0; j < PW; ++j)
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4 *>(red + (size_t)(wave * RT + 32 * j + l32) * PITCH + 32 * i + 8 * q + 4 * half) =
                    make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    __syncthreads();
    const float pad = (float)a.pad;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int idx = tid + p * 64 * KW;
        if (OUTS % (64 * KW) != 0 && idx >= OUTS) break;
        const int r = idx / QUADS, fq = idx % QUADS * 4;
        float4 s = make_float4(-pad, -pad, -pad, -pad);
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const float4 t = *reinterpret_cast<const float4 *>(red + (size_t)(k * RT + r) * PITCH + fq);
            s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
        const int row = n0 + r, f = f0 + fq;
        if (row >= a.n) continue;
        const size_t o = (size_t)row * a.k_out + f;
        const float v[4] = {s.x * Kr[p] * al[p][0], s.y * Kr[p] * al[p][1], s.z * Kr[p] * al[p][2], s.w * Kr[p] * al[p][3]};
        if ((a.k_out & 3) == 0) {                                  // (whole quads, aligned)
            if (f < a.k_out) *reinterpret_cast<float4 *>(a.out + o) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (f + q < a.k_out) a.out[o + q] = v[q];
        }
        if (a.dot_out) {
            const float d[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (f + q < a.k_out) a.dot_out[o + q] = (int32_t)d[q];
        }
    }
}

template <int FW, int PW, int KW>
static xnor_status launch_tile(LinearWordsArgs a, hipStream_t stream)
{
    constexpr size_t lds = (size_t)KW * 32 * PW * (32 * FW + 4) * sizeof(float);
    auto kern = linear_words_kernel<FW, PW, KW>;
    if (lds > 48 * 1024) {
        static std::atomic<bool> done;               // false -> true only; a repeated attribute call is harmless
        if (!done.load(std::memory_order_acquire)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
                return XNOR_ERR_HIP;
            done.store(true, std::memory_order_release);
        }
    }
    a.ptiles = (a.n + 32 * PW - 1) / (32 * PW);
    a.ftiles = (a.k_out + 32 * FW - 1) / (32 * FW);
    a.wmajor = a.ftiles >= 8;
    const long long wgs = (long long)(a.wmajor ? (a.ftiles + 7) / 8 * 8 : a.ftiles) * a.ptiles;
    if (wgs > 0x7fffffffLL) return XNOR_ERR_UNSUPPORTED;
    kern<<<dim3((unsigned)wgs), dim3(64 * KW), lds, stream>>>(a);
    return hip_status(hipGetLastError());
}

xnor_status launch_linear_words(const uint32_t *xbits, const uint32_t *words, const float *Krow, const float *alpha, float *out,
                                int32_t *dot_out, const ConvGeom &g, hipStream_t stream)
{
    const LinearWordsArgs a{xbits, words, Krow, alpha, out, dot_out, g.n, g.cw, g.k_out, g.fblocks, 32 * g.cw - g.c, 0, 0, 0};
    const LinearWordsTile t = linear_words_tile(g.n, g.k_out);
    if (t.filters == 1) return launch_tile<1, 1, 8>(a, stream);
    if (t.rows == 1) return launch_tile<2, 1, 8>(a, stream);
    return launch_tile<2, 2, 8>(a, stream);
}

}  // namespace xnor
