// Binary convolution on the matrix cores (sec. 3.2).  The +-1 product-sum that XNOR + bitcount
// evaluates is the same integer as a dot product of the sign tensors with 0 at padded positions,
// so the convolution is run as an implicit GEMM
//     D[filter][pixel] = sum_{tap, channel} sW[filter][tap][channel] * sI[pixel + tap][channel]
// followed by the fused scaling by K and alpha.  Two operand encodings, same kernel:
//   I8: signs widened to int8 (+1, -1, 0), v_mfma_i32_32x32x32_i8, int32 accumulation;
//   F4: signs widened to 4-bit floats (E2M1 codes 0x2 = +1, 0xA = -1, 0x0 = 0),
//       v_mfma_scale_f32_32x32x64_f8f6f4 with unit scales.  Products are +-1 or 0 and the sums
//       stay far below 2^24, so the float accumulation is exact.
//
// Work split: a workgroup owns FT = 32*FW*WF filters x PT = 32*PW*WP consecutive output pixels
// (pixels flattened over image, row, column so small images still fill the tile).  Per channel
// chunk it widens the packed activation bits of the input rows its pixels touch (halo included,
// halo = 0) into LDS once; every tap then reads the same LDS image at a shifted offset.
// Weights: 4-bit operands are widened in the K loop from the packed words (WStreamBits: 256 bytes per K-step and 32
// filters, seven vector instructions that hide behind the matrix instructions of the step before); the other formats read
// the pre-widened image written by the weight packer, one contiguous KiB per 32-filter operand.  Both are
// prefetched several K-steps ahead in registers.  Filters are the M operand
// and pixels the N operand, so each lane of the result holds one pixel column: stores along a
// filter plane are contiguous across lanes.
#pragma once
#include "mfma_common.h"
#include "mfma_launch.h"
#include <algorithm>
#include <atomic>
#include <type_traits>

namespace xnor {

// Sum of a KH x KW window of the staged matrix A (row pitch `pitch` floats), taps added in row-major order
// starting from +0: every read is issued before the first addition.
template <int KH, int KW> __device__ __forceinline__ float box_sum_lds(const float *ap, int pitch)
{
    float a[KH * KW];
#pragma unroll
    for (int dy = 0; dy < KH; ++dy)
#pragma unroll
        for (int dx = 0; dx < KW; ++dx) a[dy * KW + dx] = ap[dy * pitch + dx];
    float s = 0.0f;
#pragma unroll
    for (int t = 0; t < KH * KW; ++t) s += a[t];
    return s;
}

// Everything a convolution kernel is given.  One struct, so that its place in the kernel argument segment is known: a phase of
// the kernel reads the fields it needs again from there (reload) instead of holding all phases' fields in scalar registers,
// which the compiler would otherwise park in vector register lanes (two vector instructions per field and wave).
struct ConvArgs {
    const uint32_t *xbits;
    const v4i *wimg;
    const float *K, *A, *alpha;
    float *out;
    int32_t *dot_out;
    uint32_t wimg_bytes;
    ConvGeom g;
    MfmaPlan pl;
    FuseArgs fz;
};

// A fresh copy of the kernel's arguments: only the fields that are used afterwards are loaded, by scalar loads.  For plain values and for
// pointers that become buffer resources: behind a pointer read this way the compiler no longer knows global memory.
__device__ __forceinline__ ConvArgs reload_args()
{
    typedef const __attribute__((address_space(4))) uint64_t *seg_t;
    seg_t p = (seg_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));           // the compiler must not find the earlier loads' values behind it
    static_assert(sizeof(ConvArgs) % 8 == 0, "copied by 64-bit words");
    struct Words { uint64_t w[sizeof(ConvArgs) / 8]; } words;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(ConvArgs) / 8); ++i) words.w[i] = p[i];
    return __builtin_bit_cast(ConvArgs, words);
}

// What bounds it: with a few waves per SIMD every phase costs its instructions (5.2 cycles each for a wave, 4 for the SIMD);
// the K loop then runs at the matrix pipes' 32 busy cycles per instruction and SIMD (19 ns by stamps around the loop, that is
// a clock of about 1.7 GHz while all pipes are busy), which up to four vector instructions per matrix instruction do not slow down.
// Against 4-bit records in memory, a staging loop of one word per item and one set of arguments held throughout (launches
// back to back, the two in turn): 256 rows x 9216 -> 4096 14.3 -> 12.8 us, 128 x 28 x 28 batch 256 30.4 -> 26.0 us (983 -> 653
// vector instructions per wave), 96 x 27 x 27 5 x 5 batch 64 21.6 -> 20.6, 384 x 13 x 13 -> 256 batch 128 17.1 -> 15.9, 512 x 7 x 7
// batch 256 22.7 -> 21.3, 256 x 14 x 14 batch 256 23.8 -> 22.6 us.
//
// Device memory behind a pointer out of the argument struct.  Without the address space such accesses are flat ones, which
// also wait for, and are waited for with, the LDS accesses in flight.
template <class T> using global_t = __attribute__((address_space(1))) T;
template <class T> __device__ __forceinline__ global_t<T> *in_global(T *p) { return (global_t<T> *)p; }

// Accumulator tiles of up to 8 result blocks leave room for two waves per SIMD (256 registers each).
// KS > 1: KS groups of WF x WP waves share the K loop of the same tile (group k takes the k-th run of steps) and add
// their accumulators through LDS at the end: more weight loads in flight and more waves for the staging where a
// problem offers few output tiles and a long K (fully connected layers).  Consecutive-record streams only.
template <int FMT, int FW, int PW, int WF, int WP, bool FUSE, bool LINEAR, bool POOL = false, int KS = 1, bool DIRECT_CHUNKS = false>
__global__ __launch_bounds__(64 * WF * WP * KS, (FW * PW <= (FMT == 2 || FMT == 4 || FMT == 6 ? 6 : 8) && WF * WP * KS <= 8 ? 2 : 1)) void conv_mfma_kernel(
    ConvArgs args)
{
    const uint32_t *xbits = args.xbits;
    const v4i *wimg = args.wimg;
    const float *K = args.K, *A = args.A, *alpha = args.alpha;
    const uint32_t wimg_bytes = args.wimg_bytes;
    const ConvGeom &g = args.g;
    const MfmaPlan &pl = args.pl;
    const FuseArgs &fz = args.fz;
    typedef Enc<FMT> E;
    // operands staged as they are (no sign bits to widen, no K): bfloat16 parts and int8 levels
    constexpr bool RAW = FMT >= 2;
    // packed bits staged through set_direct_staging's plan
    constexpr bool DIRECT = (LINEAR || DIRECT_CHUNKS) && !RAW;
    constexpr bool ONE = LINEAR && !RAW;        // ... and one chunk holds every channel word
    static_assert(!DIRECT_CHUNKS || (FMT == 1 && !LINEAR), "chunks of packed words");
    typedef typename E::acc_t acc_t;
    static_assert(KS == 1 || (LINEAR && !FUSE && !POOL), "waves along K: plain epilogue, consecutive records");
    constexpr int NT = 64 * WF * WP * KS;
    constexpr int FT = 32 * FW * WF;
    constexpr int PT = 32 * PW * WP;
    // Weight prefetch depth.  Five steps pay off on long K loops; the 64-filter tiles serve layers
    // with short K loops and many workgroups, and the fused epilogue needs registers of its own:
    // there three steps keep more waves resident.
    // (Packed words cost one register per step: five steps throughout.)
    // A wave tile of a single result block (fully connected layers: few output tiles, long K) issues one matrix
    // instruction per record: only a deep ring keeps enough bytes in flight to cover the L2 latency.
    constexpr int DW = FMT == 2 || FMT == 4 || FMT == 6 ? 3 : (FW * PW == 1 && FMT < 2 && !FUSE) ? 7 : (FMT == 1) ? 5 : (FUSE || FT <= 64) ? 3 : 5;      // (bfloat16 parts: a step is three times as long)
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    int *rowinfo = reinterpret_cast<int *>(lds + pl.region_bytes);
    int *xoff_tab = rowinfo + pl.max_rows;     // [(nsteps + KLOOP_TABLE_PAD) * BPS]
    float *a_lds = reinterpret_cast<float *>(xoff_tab + (pl.nsteps + KLOOP_TABLE_PAD) * E::BPS);   // [max_rows * wp], halo = 0
    float *ktile = a_lds + pl.max_rows * g.wp;                                   // [PT]
    float *asum_lds = ktile + PT;                                                // [WF][PT], fused epilogue only
    uint32_t *wtile_lds = reinterpret_cast<uint32_t *>(asum_lds + WF * PT);      // [PT][FT/32], fused epilogue only
    // sign byte -> operand bytes table, after everything else (16-byte aligned by the plan)
    const uint8_t *lut = lds + pl.lut_offset;

    // Workgroups go to the 8 XCDs round-robin by (linear) index, and every XCD has its own L2.
    //  - Usual case (activations outweigh weights): within every window of 64 pixel tiles each XCD
    //    takes a run of 8 consecutive ones, so that the output lines two neighbouring tiles both
    //    write in part (and the input rows they share) meet in one XCD's L2.  The last, incomplete
    //    window keeps the plain order: runs would load the XCDs unevenly there.
    //  - Weight-heavy problems (fully connected layers): all pixel tiles of one filter tile go to
    //    one XCD, so that each XCD fetches only its own filter tiles' weights from HBM instead of
    //    all eight fetching everything.  1-D grid: XCD = index % 8, filter tile = 8 * (slot /
    //    ptiles) + XCD, pixel tile = slot % ptiles, slot = index / 8.
    uint32_t ptile, ftile;
    if (pl.wmajor) {
        const uint32_t xcd = blockIdx.x & 7u, slot = blockIdx.x >> 3;
        ftile = (slot / (uint32_t)pl.ptiles) * 8u + xcd;
        ptile = slot % (uint32_t)pl.ptiles;
        if (ftile >= (uint32_t)pl.ftiles) return;
    } else {
        const uint32_t bx = blockIdx.x;
        const uint32_t win = (bx >> 6) << 6;
        ptile = win + 64u <= (uint32_t)pl.ptiles ? win + ((bx & 7u) << 3) + ((bx >> 3) & 7u) : bx;
        ftile = blockIdx.y;
        if (ptile >= (uint32_t)pl.ptiles) return;
    }
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int l32 = lane & 31, half = lane >> 5;
    const int wk = wave / (WF * WP);                  // the wave's run of K-steps (0 without waves along K)
    const int wf = (wave % (WF * WP)) % WF, wp = (wave % (WF * WP)) / WF;
    const int f0 = (int)ftile * FT;
    const uint32_t howo = (uint32_t)(g.ho * g.wo);
    // the tile's run of flattened output pixels [m0, m_end): PT consecutive ones, or (pooled epilogue) the
    // convolution rows under a group of pooled rows of one image
    uint32_t m0, m_end;
    uint32_t pool_img = 0;
    int pool_py0 = 0, pool_rows = 0;               // first pooled row and pooled rows of this tile
    if constexpr (POOL) {
        pool_img = pl.pool.div_groups.div(ptile);
        const int gi = (int)(ptile - pool_img * (uint32_t)pl.pool.groups);
        pool_py0 = gi * pl.pool.pr;
        pool_rows = min(pl.pool.pr, pl.pool.hpo - pool_py0);
        m0 = pool_img * howo + (uint32_t)(pool_py0 * pl.pool.sh * g.wo);
        m_end = m0 + (uint32_t)(((pool_rows - 1) * pl.pool.sh + pl.pool.ph) * g.wo);
    } else {
        m0 = ptile * (uint32_t)PT;
        m_end = min(m0 + (uint32_t)PT, (uint32_t)g.m_total);
    }
    const int ccw = pl.cc_words;
    const int nsteps = pl.nsteps;

    // padded input rows this tile touches: R = image*hp + padded row
    const uint32_t m_last = m_end - 1u;
    const uint32_t img_a = g.div_howo.div(m0), img_b = g.div_howo.div(m_last);
    const uint32_t oy_a = g.div_wo.div(m0 - img_a * howo), oy_b = g.div_wo.div(m_last - img_b * howo);
    const int r_lo = (int)(img_a * g.hp + oy_a * g.sh);
    const int r_hi = (int)(img_b * g.hp + oy_b * g.sh) + g.kh - 1;
    const int nrows = r_hi - r_lo + 1;

    // alpha (fused epilogue: also scale and shift) of this workgroup's filters: requested first, written behind the widening
    // table ([FT] each), raw operands at once, the others when the staging loads are on their way; filters past the last one
    // repeat it and are masked later
    constexpr int NP = (FT + NT - 1) / NT;
    float par[NP][FUSE ? 3 : 1];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int kc = min(f0 + tid + u * NT, g.k_out - 1);
        par[u][0] = in_global(alpha)[kc];
        if constexpr (FUSE) {
            par[u][1] = fz.bn_scale ? in_global(fz.bn_scale)[kc] : 1.0f;
            par[u][2] = fz.bn_scale ? in_global(fz.bn_shift)[kc] : 0.0f;
        }
    }
    float *par_lds = reinterpret_cast<float *>(lds + pl.lut_offset + E::LUT_BYTES);
    E::build_lut(lds + pl.lut_offset, tid, NT);
    auto store_par = [&] {
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (NP * NT == FT || tid + u * NT < FT) {
                par_lds[tid + u * NT] = par[u][0];
                if constexpr (FUSE) {
                    par_lds[FT + tid + u * NT] = par[u][1];
                    par_lds[2 * FT + tid + u * NT] = par[u][2];
                }
            }
    };
    if constexpr (RAW) store_par();
    if constexpr (!DIRECT)
    for (int rr = tid; rr < nrows; rr += NT) {
        const uint32_t R = (uint32_t)(r_lo + rr);
        const uint32_t img = pl.div_hp.div(R);
        const int y = (int)(R - img * g.hp) - g.ph;
        // first pixel of the (real) input row, -1 for padding rows and the zero rows of a dilated input
        const uint32_t ry = g.div_dil_h.div_small((uint32_t)max(y, 0));
        const bool rv = y >= 0 && y < g.h && (int)ry * g.dil_h == y && (int)ry < g.real_h;
        rowinfo[rr] = rv ? (int)((img * g.real_h + ry) * g.real_w) : -1;
    }
    // LDS offset of every channel block of a chunk relative to a pixel's window origin:
    // block b = tap * ccw + word  ->  (dy*wp + dx)*ps + word*BPB
    {
        const int nblk = g.taps * ccw;
        for (int b = tid; b < (nsteps + KLOOP_TABLE_PAD) * E::BPS; b += NT) {     // padding repeats the last block
            const uint32_t bb = (uint32_t)min(b, nblk - 1);
            const uint32_t t = pl.div_ccw.div_small(bb);
            const uint32_t wl = bb - t * ccw;
            const uint32_t dy = g.div_kw.div_small(t);
            const uint32_t dx = t - dy * g.kw;
            xoff_tab[b] = (int)(dy * pl.row_pitch + dx * pl.ps + wl * E::BPB);
        }
    }
    // pixel t of the tile: image (counted from img_a), padded row (from r_lo) and column of its window's origin
    const uint32_t rel0 = m0 - img_a * howo;
    auto locate = [=](const ConvGeom &g, const MfmaPlan &pl, uint32_t t, uint32_t &img, uint32_t &pix, int &row, int &col) {
        const uint32_t rel = rel0 + min(t, m_end - 1u - m0);
        uint32_t oy, ox;
        if constexpr (DIRECT) {
            const uint32_t rows = pl.sd_wo.div(rel);
            img = pl.sd_ho.div(rows);
            oy = rows - mul24(img, (uint32_t)g.ho);
            ox = rel - mul24(rows, (uint32_t)g.wo);
            pix = rel - mul24(img, (uint32_t)(g.ho * g.wo));
        } else {
            const uint32_t howo = (uint32_t)(g.ho * g.wo);
            img = g.div_howo.div(rel);
            pix = rel - img * howo;
            oy = g.div_wo.div(pix);
            ox = pix - oy * g.wo;
        }
        row = (int)(img * g.hp + (oy - oy_a) * g.sh);
        col = (int)ox * g.sw;
    };
    // LDS byte offset of each of this lane's pixel columns (window origin in the padded frame)
    int pbase[PW];
#pragma unroll
    for (int j = 0; j < PW; ++j) {
        uint32_t img, pix;
        int row, col;
        locate(g, pl, (uint32_t)((wp * PW + j) * 32 + l32), img, pix, row, col);
        pbase[j] = row * pl.row_pitch + col * pl.ps + (E::HALF_SPLIT ? 16 * half : 0);
    }
    // weight records of this wave's filter blocks: record index = fblk * recs_per_fblock + step record
    const int recs_per_fb = (g.taps * g.cw + E::BPS - 1) / E::BPS;
    // Weight records are fetched with buffer loads: scalar record offset + the lane's 16-byte slot,
    // so the K loop spends no vector registers or ALU work on weight addresses.
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<v4i *>(wimg), 0, (int)wimg_bytes, 0x00020000);
    const int wlane = lane * 16;
    const int zero_rec = (int)(wimg_bytes >> 10) - 1;      // the image ends with an all-zero record
    int wrec0[FW];
#pragma unroll
    for (int i = 0; i < FW; ++i) {
        const int fb = min(f0 / 32 + wf * FW + i, g.fblocks - 1);
        wrec0[i] = __builtin_amdgcn_readfirstlane(fb * recs_per_fb);
    }
    const int tab_lane = (E::HALF_SPLIT ? 0 : half);

    acc_t acc[FW][PW];
#pragma unroll
    for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int j = 0; j < PW; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
    const int steps_per_tap = pl.tap_jump ? max(ccw / E::BPS, 1) : 0x7fffffff;
    for (int wbase = 0; ONE ? wbase < 1 : wbase < args.g.cw; wbase += ONE ? 1 : ccw) {
        // (read per chunk: otherwise everything a chunk derives from them is hoisted in front of the first one and held.  Raw
        // operands hold little: there the loads cost more, 4 images of 32x12x12 -> 497, 1x1, int8 levels 4.6 us with them, 4.3 without)
        const ConvArgs now = RAW ? args : reload_args();
        const ConvGeom &g = now.g;
        const MfmaPlan &pl = now.pl;
        const v4i *wimg = now.wimg;
        // packed weight words, widened in the K loop: the first steps' are requested ahead of the staging, which hides their latency
        // (a register per step and filter block; requested behind it, 100 layers of 16 to 512 channels took 1.006 of the time in the mean, fused 1.001)
        constexpr bool WORDS = FMT == 1 || FMT == 2;
        const int per = (nsteps + KS - 1) / KS;
        const int s0 = KS > 1 ? __builtin_amdgcn_readfirstlane(wk * per) : 0;
        const int ns = KS > 1 ? max(0, min(per, nsteps - s0)) : nsteps;
        auto words_of = [&] {
            int fblk[FW];
#pragma unroll
            for (int i = 0; i < FW; ++i)
                fblk[i] = __builtin_amdgcn_readfirstlane(min(f0 / 32 + wf * FW + i, g.fblocks - 1));
            const bool odd = (g.taps * ccw) % 2 != 0 && s0 + ns == nsteps;
            return WStreamBits<FW, LINEAR, KS != 1 ? 2 : 0>(reinterpret_cast<const uint32_t *>(wimg), fblk, g.taps * g.cw,
                                                            wbase + s0 * E::BPS, ns, odd, lane, steps_per_tap, pl.tap_jump,
                                                            FMT == 2 && ccw == 1 ? g.cw : 1);
        };
        typedef typename std::conditional<WORDS, uint32_t, v4i>::type weight_t;
        weight_t w[DW + 1][FW];
        typename std::conditional<WORDS, WStreamBits<FW, LINEAR, KS != 1 ? 2 : 0>, int>::type words{};
        if constexpr (WORDS) {
            words = words_of();
#pragma unroll
            for (int u = 0; u < DW; ++u) words.load(w[u]);
        }
        if (wbase > 0 || !ONE || E::LUT_BYTES > 0) __syncthreads();   // tables visible / previous chunk fully consumed
        const bool stageA = !RAW && wbase == 0 && !K;
        if constexpr (DIRECT) {
            const int px_a = g.real_h * g.real_w;
            const uint32_t left = (uint32_t)(g.n - (int)img_a) * (uint32_t)px_a;       // (validated: n * h * w fits 31 bits)
            // (the images a tile can touch stay below 2 GiB; the resource may end early, never late)
            const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint32_t *>(xbits) + (size_t)img_a * px_a * g.cw, 0,
                (int)min((size_t)left * (uint32_t)g.cw * 4u, (size_t)0x7ffffff0), 0x00020000);
            const __amdgpu_buffer_rsrc_t arsrc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float *>(A) + (size_t)img_a * px_a, 0, stageA ? (int)(min(left, 0x1fffffffu) * 4u) : 0, 0x00020000);
            const int items = nrows * g.wp * pl.quads;
            const int y0 = (int)oy_a * g.sh;
            auto stage = [&](auto vecc, auto dilc) {
                constexpr int V = decltype(vecc)::value;
                constexpr bool DILATED = decltype(dilc)::value;
                constexpr int FB = 4;           // items in flight per thread: a tile rarely has more
                for (int base = 0; base < items; base += NT * FB) {
                    uint32_t bits[FB][V];
                    float av[FB];
                    int dst[FB], adst[FB], wl[FB];
                    bool ok[FB];
#pragma unroll
                    for (int u = 0; u < FB; ++u) {
                        if (base + u * NT >= items) break;                              // (uniform)
                        const uint32_t it = (uint32_t)(base + u * NT + tid);
                        const uint32_t px = pl.sd_quads.div(it), q = it - mul24(px, (uint32_t)pl.quads);
                        // first word of the item's load
                        const uint32_t w0 = ONE && V == 4 ? min(q * V, (uint32_t)(pl.cc_words - V)) : q * V;
                        const uint32_t rr = pl.sd_wp.div(px);
                        const uint32_t xc = px - mul24(rr, (uint32_t)g.wp);
                        const uint32_t yy = (uint32_t)y0 + rr, img = pl.sd_hp.div(yy);
                        uint32_t y = yy - mul24(img, (uint32_t)g.hp) - (uint32_t)g.ph, x = xc - (uint32_t)g.pw;
                        ok[u] = (int)it < items && y < (uint32_t)g.h && x < (uint32_t)g.w;
                        if constexpr (DILATED) {       // zeros between the real pixels and beyond the last ones
                            const uint32_t yr = pl.sd_dil_h.div(y), xr = pl.sd_dil_w.div(x);
                            ok[u] = ok[u] && mul24(yr, (uint32_t)g.dil_h) == y && mul24(xr, (uint32_t)g.dil_w) == x &&
                                    yr < (uint32_t)g.real_h && xr < (uint32_t)g.real_w;
                            y = yr;
                            x = xr;
                        }
                        const uint32_t pix = mul24(mul24(img, (uint32_t)g.real_h) + y, (uint32_t)g.real_w) + x;
                        const uint32_t off = ok[u] ? mul24(pix, (uint32_t)g.cw * 4u) + w0 * 4u + (ONE ? 0u : (uint32_t)wbase * 4u) : 0x80000000u;
                        if constexpr (V == 4) {
                            const v4u r = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)off, 0, 0);
                            bits[u][0] = r[0]; bits[u][1] = r[1]; bits[u][2] = r[2]; bits[u][3] = r[3];
                        } else if constexpr (V == 3) {
                            const auto r = __builtin_amdgcn_raw_buffer_load_b96(xrsrc, (int)off, 0, 0);
                            bits[u][0] = r[0]; bits[u][1] = r[1]; bits[u][2] = r[2];
                        } else if constexpr (V == 2) {
                            const auto r = __builtin_amdgcn_raw_buffer_load_b64(xrsrc, (int)off, 0, 0);
                            bits[u][0] = r[0]; bits[u][1] = r[1];
                        } else {
                            bits[u][0] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (int)off, 0, 0);
                        }
                        wl[u] = (ONE ? 0 : wbase) + (int)w0;
                        const bool first = stageA && q == 0 && (int)it < items;
                        adst[u] = first ? (int)px : -1;
                        if (stageA)
                            av[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                                  arsrc, (int)(ok[u] && q == 0 ? pix * 4u : 0x80000000u), 0, 0));
                        dst[u] = (int)it < items ? (int)(mul24(rr, (uint32_t)pl.row_pitch) + mul24(xc, (uint32_t)pl.ps) +
                                                         w0 * (uint32_t)E::BPB)
                                                 : -1;
                    }
#pragma unroll
                    for (int u = 0; u < FB; ++u) {
                        if (base + u * NT >= items) break;
                        if (dst[u] >= 0) {
#pragma unroll
                            for (int v = 0; v < V; ++v) {
                                const int nch = g.c % 32 == 0 ? 32 : g.c - (wl[u] + v) * 32;
                                E::widen_word_lut(lds + dst[u] + v * E::BPB, lut, bits[u][v],
                                                  ok[u] && (ONE || wl[u] + v < g.cw), nch);
                            }
                            if (stageA && adst[u] >= 0) a_lds[adst[u]] = av[u];
                        }
                    }
                }
            };
            auto by_width = [&](auto dilated) {
                if (pl.vec == 4) stage(std::integral_constant<int, 4>{}, dilated);
                else if (pl.vec == 3) stage(std::integral_constant<int, 3>{}, dilated);
                else if (pl.vec == 2) stage(std::integral_constant<int, 2>{}, dilated);
                else stage(std::integral_constant<int, 1>{}, dilated);
            };
            // (dilated inputs: backward convolutions, which have the plain epilogue)
            if (!FUSE && !POOL && pl.dilated) by_width(std::bool_constant<!FUSE && !POOL>{});
            else by_width(std::false_type{});
        } else {
        const int items = nrows * g.wp * ccw;
        if constexpr (FMT == 2) {
            if (g.stored_digits) {
                // digits as the split wrote them: 16 of a word's 128 bytes per item, a pixel's words of the chunk one after the other
                constexpr int FB = 4;          // items in flight per thread
                const int units = items * 8;
                for (int it0 = tid; it0 < units; it0 += NT * FB) {
                    v4u d[FB];
                    int dst[FB];
#pragma unroll
                    for (int u = 0; u < FB; ++u) {
                        const int it = it0 + u * NT;
                        const uint32_t item = (uint32_t)min(it, units - 1) >> 3, unit = (uint32_t)it & 7u;
                        const uint32_t px = pl.div_ccw.div_small(item);
                        const int wl = (int)(item - px * ccw);
                        const uint32_t rr = pl.div_wp.div_small(px);
                        const int xcol = (int)(px - rr * g.wp) - g.pw;
                        const int rowbase = rowinfo[rr];
                        const bool ok = rowbase >= 0 && xcol >= 0 && xcol < g.w && wbase + wl < g.cw;
                        dst[u] = it < units ? (int)(rr * pl.row_pitch + (px - rr * g.wp) * pl.ps + wl * E::BPB + unit * 16) : -1;
                        const uint32_t word = ok ? (uint32_t)(rowbase + xcol) * (uint32_t)g.cw + (uint32_t)(wbase + wl) : 0u;
                        d[u] = in_global(reinterpret_cast<const v4u *>(xbits))[(size_t)word * 8 + unit];
                        if (!ok) d[u] = v4u{0, 0, unit == 7u ? 127u : 0u, 0};
                    }
#pragma unroll
                    for (int u = 0; u < FB; ++u)
                        if (dst[u] >= 0) *reinterpret_cast<v4u *>(lds + dst[u]) = d[u];
                }
            } else {
            // 32 channels of a pixel per item: two groups of three bfloat16 parts (192 bytes), summed back to floats (exact),
            // to digits
            const int groups = (g.c + 15) / 16;
            for (int it = tid; it < items; it += NT) {
                const uint32_t px = pl.div_ccw.div_small((uint32_t)it);
                const int wl = it - (int)px * ccw;
                const uint32_t rr = pl.div_wp.div_small(px);
                const int xcol = (int)(px - rr * g.wp) - g.pw;
                const int rowbase = rowinfo[rr];
                const int grp = 2 * (wbase + wl);
                const bool ok = rowbase >= 0 && xcol >= 0 && xcol < g.w && grp < groups;
                v4u *dst = reinterpret_cast<v4u *>(lds + rr * pl.row_pitch + (px - rr * g.wp) * pl.ps + wl * E::BPB);
                if (!ok) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) dst[q] = v4u{0, 0, q == 7 ? 127u : 0u, 0};
                    continue;
                }
                const auto *src = in_global(reinterpret_cast<const v4u *>(xbits)) + (((size_t)rowbase + xcol) * groups + grp) * 6;
                v4u p[12];
#pragma unroll
                for (int q = 0; q < 6; ++q) p[q] = src[q];
                const int second = grp + 1 < groups ? 6 : 0;      // (no second group: the first one again, cleared below)
#pragma unroll
                for (int q = 0; q < 6; ++q) p[6 + q] = src[second + q];
                float x[32];
#pragma unroll
                for (int c = 0; c < 32; ++c) {
                    auto part = [&](int k) {
                        const uint32_t d = p[6 * (c / 16) + 2 * k + c % 16 / 8][c % 8 / 2];
                        return __builtin_bit_cast(float, c % 2 ? d & 0xffff0000u : d << 16);
                    };
                    x[c] = part(0) + (part(1) + part(2));
                    if (c >= 16) x[c] = second ? x[c] : 0.0f;
                }
                uint32_t out[32];
                E::digits(x, out);
#pragma unroll
                for (int q = 0; q < 8; ++q) dst[q] = v4u{out[4 * q], out[4 * q + 1], out[4 * q + 2], out[4 * q + 3]};
            }
            }
        } else if constexpr (FMT == 6) {
            // the three parts of 16 channels of a pixel per item, from their half of a word of digits
            const int cg = ccw / 3, words = (g.cw / 3 + 1) / 2;
            for (int it = tid; it < items / 3; it += NT) {
                const int px = it / cg, grp = wbase / 3 + it - px * cg;
                const uint32_t rr = pl.div_wp.div_small((uint32_t)px);
                const int xcol = px - (int)rr * g.wp - g.pw;
                const int rowbase = rowinfo[rr];
                v4u parts[6] = {};
                if (rowbase >= 0 && xcol >= 0 && xcol < g.w) {
                    const auto *src = in_global(reinterpret_cast<const v4u *>(xbits)) + (((size_t)rowbase + xcol) * words + grp / 2) * 8;
                    v4u word[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) word[q] = src[q];
                    E::parts_of_digits(word, grp & 1, parts);
                }
                v4u *dst = reinterpret_cast<v4u *>(lds + rr * pl.row_pitch + (px - (int)rr * g.wp) * pl.ps + (it - px * cg) * 3 * E::BPB);
#pragma unroll
                for (int q = 0; q < 6; ++q) dst[q] = parts[q];
            }
        } else {
        constexpr int FB = RAW ? 4 : 8;        // items in flight per thread: loads first, then widening (every batch costs one round trip to L2 or HBM)
        for (int it0 = tid; it0 < items; it0 += NT * FB) {
            uint32_t bits[FB];
            v4u raw[FB][2];                // (raw operands: the 32-byte word itself)
            int dst[FB], nch[FB];
            bool ok[FB];
#pragma unroll
            for (int u = 0; u < FB; ++u) {
                const int it = it0 + u * NT;
                const uint32_t itc = (uint32_t)min(it, items - 1);
                const uint32_t px = pl.div_ccw.div_small(itc);
                const int wl = (int)(itc - px * ccw);
                const uint32_t rr = pl.div_wp.div_small(px);
                const int xv = (int)(px - rr * g.wp) - g.pw;                 // column of the (virtual) input
                const int xcol = (int)g.div_dil_w.div_small((uint32_t)max(xv, 0));  // column of the real tensor
                const int rowbase = rowinfo[rr];
                // (only packed words have a last chunk that may lack one)
                ok[u] = rowbase >= 0 && xv >= 0 && xv < g.w && xcol * g.dil_w == xv && xcol < g.real_w && (FMT != 1 || wbase + wl < g.cw);
                dst[u] = it < items ? (int)(rr * pl.row_pitch + (px - rr * g.wp) * pl.ps + wl * E::BPB) : -1;
                nch[u] = g.c - (wbase + wl) * 32;
                bits[u] = 0;
                if constexpr (RAW) {
                    raw[u][0] = raw[u][1] = v4u{0, 0, 0, 0};
                    if (ok[u]) {
                        const auto *src = in_global(reinterpret_cast<const v4u *>(xbits)) +
                                          (((size_t)rowbase + xcol) * g.cw + wbase + wl) * 2;
                        raw[u][0] = src[0];
                        raw[u][1] = src[1];
                    }
                } else {
                    if (ok[u]) bits[u] = in_global(xbits)[((size_t)rowbase + xcol) * g.cw + wbase + wl];
                }
            }
#pragma unroll
            for (int u = 0; u < FB; ++u)
                if (dst[u] >= 0) {
                    if constexpr (FMT == 5) {
                        *reinterpret_cast<v4i *>(lds + dst[u]) = ok[u] ? E::narrow(raw[u][0], raw[u][1]) : v4i{0, 0, 0, 0};
                    } else if constexpr (RAW) {
                        *reinterpret_cast<v4u *>(lds + dst[u]) = raw[u][0];
                        *reinterpret_cast<v4u *>(lds + dst[u] + 16) = raw[u][1];
                    } else {
                        E::widen_word_lut(lds + dst[u], lut, bits[u], ok[u], nch[u]);
                    }
                }
        }
        }
        }
        if (!DIRECT && stageA) {
            // the matrix A of the same input rows (0 in the halo), for the K of this tile
            for (int it = tid; it < nrows * g.wp; it += NT) {
                const uint32_t rr = pl.div_wp.div_small((uint32_t)it);
                const int xcol = it - (int)rr * g.wp - g.pw;
                const int rowbase = rowinfo[rr];
                a_lds[it] = rowbase >= 0 && xcol >= 0 && xcol < g.w ? in_global(A)[(size_t)rowbase + xcol] : 0.0f;
            }
        }
        if (!RAW && wbase == 0) store_par();
        __syncthreads();
        // K of the tile's output pixels, an equal share per wave: the kh x kw taps of A in row-major order over the
        // staged rows (halo entries add +0.0f, the same bits as skipping them), divided by kh*kw
        constexpr int KPW = (PT + WF * WP * KS - 1) / (WF * WP * KS);
        if (!RAW && wbase == 0 && !K) for (int kt = wave * KPW + lane; kt < min((wave + 1) * KPW, PT); kt += 64) {
            uint32_t img, pix;
            int row, col;
            locate(g, pl, (uint32_t)kt, img, pix, row, col);
            const float *ap = a_lds + row * g.wp + col;
            // the common filters with every tap's read in flight at once (one LDS latency instead of one per group
            // of four taps); the additions keep the row-major order either way
            float s;
            if (g.kh == 3 && g.kw == 3) s = box_sum_lds<3, 3>(ap, g.wp);
            else if (g.kh == 5 && g.kw == 5) s = box_sum_lds<5, 5>(ap, g.wp);
            else if (g.kh == 1 && g.kw == 1) s = 0.0f + ap[0];
            else {
                s = 0.0f;
                for (int dy = 0; dy < g.kh; ++dy, ap += g.wp)
                    for (int dx0 = 0; dx0 < g.kw; dx0 += 4) {
                        float a[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) a[u] = ap[min(dx0 + u, g.kw - 1)];
#pragma unroll
                        for (int u = 0; u < 4; ++u) s += dx0 + u < g.kw ? a[u] : 0.0f;
                    }
            }
            ktile[kt] = s / (float)(g.kh * g.kw);
        }

        // ---- software-pipelined K loop over this chunk's steps --------------------------------
        // record of step s: rec0 + s + (s / steps_per_tap) * tap_jump
        auto request = [&](auto &ws) {
#pragma unroll
            for (int u = 0; u < DW; ++u) ws.load(w[u]);
        };
        if constexpr (FMT == 2) {
            mfma_kloop_digits<FW, PW, DW>(acc, lds, pbase, xoff_tab, tab_lane, words, w, ns);
        } else if constexpr (WORDS) {
            mfma_kloop<E, FW, PW, DW, 1>(acc, lds, pbase, xoff_tab + s0 * E::BPS, tab_lane, words, w, ns);
        } else if constexpr (LINEAR && KS > 1) {
            // (problems that take this form are all weights: an image read once per call, which passes every XCD's L2 on its
            // way and should not settle in the last-level cache: fully connected layer inside a step 27.3 -> 24.3 us)
            WStreamLinear<FW, 2> ws(wimg, wrec0, wbase / E::BPS + s0, ns, wlane);
            request(ws);
            mfma_kloop<E, FW, PW, DW, 1>(acc, lds, pbase, xoff_tab + s0 * E::BPS, tab_lane, ws, w, ns);
        } else if constexpr (LINEAR) {      // the chunk holds every channel word: consecutive records
            WStreamLinear<FW> ws(wimg, wrec0, wbase / E::BPS, nsteps, wlane);
            request(ws);
            mfma_kloop<E, FW, PW, DW, 1>(acc, lds, pbase, xoff_tab, tab_lane, ws, w, nsteps);
        } else {
            WStreamChunked<FW> ws(wrsrc, wrec0, zero_rec, wbase / E::BPS, nsteps, steps_per_tap, pl.tap_jump, wlane);
            request(ws);
            mfma_kloop<E, FW, PW, DW, 1>(acc, lds, pbase, xoff_tab, tab_lane, ws, w, nsteps);
        }
    }
    {
    const ConvArgs late = RAW ? args : reload_args();
    const ConvGeom &g = late.g;
    const MfmaPlan &pl = late.pl;
    const FuseArgs &fz = late.fz;
    float *out = late.out;
    int32_t *dot_out = late.dot_out;
    const uint32_t howo = (uint32_t)(g.ho * g.wo);
    // epilogue: out = float(dot) * K * alpha; result register v of a lane is filter row
    // 8*(v/4) + 4*half + v%4 of the 32-filter block, pixel column l32.  alpha of the lane's
    // filter rows is fetched once (clamped index, no branch), stores are predicated.
    if (!RAW && !K) __syncthreads();      // the K tile is complete
    if constexpr (KS > 1) {
        // the wave groups' partial sums (exact integers) meet in LDS, laid over the finished activation region
        // ([group - 1][wave][block][register][lane]: consecutive lanes, consecutive words); group 0 adds them in order
        __syncthreads();                  // every wave is done reading activations
        typedef typename std::remove_reference<decltype(acc[0][0][0])>::type elem_t;
        elem_t *redw = reinterpret_cast<elem_t *>(lds);
        const int slot = ((wk - 1) * WF * WP + (wave % (WF * WP))) * FW * PW;
        if (wk > 0) {
#pragma unroll
            for (int i = 0; i < FW; ++i)
#pragma unroll
                for (int j = 0; j < PW; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) redw[((slot + i * PW + j) * 16 + v) * 64 + lane] = acc[i][j][v];
        }
        __syncthreads();
        if (wk > 0) return;               // (no barrier follows in the plain epilogue)
#pragma unroll
        for (int k = 1; k < KS; ++k)
#pragma unroll
            for (int i = 0; i < FW; ++i)
#pragma unroll
                for (int j = 0; j < PW; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[i][j][v] += redw[(((k - 1) * WF * WP + wave) * FW * PW + i * PW + j) * 16 * 64 + v * 64 + lane];
    }
    uint32_t pimg[PW], ppix[PW];
    float Km[PW];
    bool plive[PW];
#pragma unroll
    for (int j = 0; j < PW; ++j) {
        const int pl_idx = (wp * PW + j) * 32 + l32;
        const uint32_t m = m0 + (uint32_t)pl_idx;
        plive[j] = m < m_end;
        int row, col;
        locate(g, pl, (uint32_t)pl_idx, pimg[j], ppix[j], row, col);
        Km[j] = 1.0f;                                 // (real and k-bit activations carry no K)
        if constexpr (!RAW) {
            if (K) Km[j] = in_global(K)[g.k_per_image ? img_a + pimg[j] : min(m, m_end - 1u)];
            else Km[j] = ktile[pl_idx];
        }
    }
    // Float (and optional integer) results leave through buffer stores: the resource starts at the
    // tile's first image, a lane's vector offset names its pixel (plus its half-wave's four rows),
    // the filter row is a scalar offset (16-byte stores: see there), so a store needs no per-lane address arithmetic.  Dead
    // pixel columns and rows past the last filter get an offset beyond the resource, which the
    // buffer bounds check discards.  (The host refuses shapes whose tile span exceeds 2 GiB.)
    const size_t img_elems = (size_t)g.k_out * howo;
    const uint32_t span = (uint32_t)min((size_t)(g.n - (int)img_a) * img_elems * 4, (size_t)0x7ffffff0);
    const uint32_t OOB = 0x80000000u;
    uint32_t voff[PW];
#pragma unroll
    for (int j = 0; j < PW; ++j)
        voff[j] = plive[j] ? (uint32_t)((pimg[j] * (uint32_t)img_elems + ppix[j] + 4u * half * howo) * 4u) : OOB;
    const int wf_s = __builtin_amdgcn_readfirstlane(wf);
    auto store_rows = [&](auto *dst, int i, int j, auto value_of) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(dst + (size_t)img_a * img_elems, 0, (int)span, 0x00020000);
        const int row0 = f0 + (wf_s * FW + i) * 32;                 // wave-uniform
        if (row0 + 32 <= g.k_out && howo == 1u && (g.k_out & 3) == 0) {
            // planes of one pixel (fully connected layers): a lane's four consecutive filter rows are 16
            // contiguous, aligned bytes.  A store of more than 64 bits still reads its data two wait states after it
            // issued; the compiler keeps the next write of those registers that far away unless the scalar offset is a
            // register, so the row goes into the vector offset (with it in the scalar one, 16 to 64 of the 280576 results
            // of 8768 rows, 5 features and 32 filters were now and then those of other filters).  The distance costs
            // 0.25 us of a launch (256 rows, 9216 -> 4096: 12.4 -> 12.65 us), as does one kept by explicit waits.
            const uint32_t v0 = voff[j] + 4u * (uint32_t)row0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                __builtin_amdgcn_raw_buffer_store_b128(v4u{value_of(4 * q), value_of(4 * q + 1), value_of(4 * q + 2),
                                                           value_of(4 * q + 3)},
                                                       rs, (int)(v0 + 32u * q), 0, 0);
            return;
        }
        // Results larger than a quarter of the 256 MB last-level cache leave with the non-temporal hint (measured: a
        // 205 MB result 59 -> 44 us, 103 MB 42 -> 32 us, while 51 MB and smaller results are 10 us slower with it).
        // The cache policy is part of the instruction: one run of stores per policy, chosen by a uniform branch.
        auto rows = [&](auto aux) {
            constexpr int AUX = decltype(aux)::value;
            if (row0 + 32 <= g.k_out) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    __builtin_amdgcn_raw_buffer_store_b32(value_of(v), rs, (int)voff[j],
                                                          (row0 + 8 * (v >> 2) + (v & 3)) * (int)howo * 4, AUX);
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = row0 + 8 * (v >> 2) + (v & 3);
                    const bool fin = row + 4 * half < g.k_out;
                    __builtin_amdgcn_raw_buffer_store_b32(value_of(v), rs, (int)(fin ? voff[j] : OOB),
                                                          min(row, g.k_out - 1) * (int)howo * 4, AUX);
                }
            }
        };
        if (pl.stream_out) rows(std::integral_constant<int, 2>{});
        else rows(std::integral_constant<int, 0>{});
    };
    if constexpr (POOL) {
    // Pooled epilogue: y = float(dot) * K * alpha (optionally max(y, 0)) of one filter block goes to a
    // per-wave LDS tile [32 filters][PT + 1 pixels] laid over the (finished) activation region; lanes
    // then take the maximum over the pooling windows and store the pooled rows of this tile.  LDS serves
    // one wave's instructions in order, so a wave's own writes are visible to its reads without a
    // workgroup barrier.  The maximum starts at -inf and skips NaN (maxNum).
    constexpr int YP = PT + 1;
    float al[FW][16];
#pragma unroll
    for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 a4 = *reinterpret_cast<const float4 *>(par_lds + (wf * FW + i) * 32 + 8 * q + 4 * half);
            al[i][4 * q] = a4.x; al[i][4 * q + 1] = a4.y; al[i][4 * q + 2] = a4.z; al[i][4 * q + 3] = a4.w;
        }
    __syncthreads();                              // every wave is done reading activations (and alpha is in registers)
    // 16 filter rows at a time (register groups v = 0..7, then 8..15): [16][PT + 1] floats per wave
    float *ystage = reinterpret_cast<float *>(lds) + (size_t)wave * 16 * YP;
    const PoolPlan &pp = pl.pool;
    const int npool = pool_rows * pp.wpo;         // pooled pixels of this tile
    // lanes -> (filter offset, pooled pixel): as many filters side by side as fit into the wave; a lane
    // keeps its pooled pixel and walks the filters in steps of nf, eight filters' window loads in flight
    const int nf = npool >= 64 ? 1 : min(64 / npool, 16);
    const int fo = npool >= 64 ? 0 : lane / npool;
    const int pq = lane - fo * npool;
    const int pstep = npool >= 64 ? 64 : npool;
    const bool lane_on = fo < nf;
    float *pooled = reinterpret_cast<float *>(out);
    const size_t plane = (size_t)pp.hpo * pp.wpo;
    // maxima of 8 filters (rows fb + u*nf + fo of the staged 16) over one pooled pixel's window
    auto window_max = [&](auto PHc, auto PWc, const float *win, const int (&roff)[8], float (&mx)[8]) {
        constexpr int CH = decltype(PHc)::value, CW = decltype(PWc)::value;       // 0: run-time window
        if constexpr (CH > 0) {
            float t[CH * CW][8];
#pragma unroll
            for (int dy = 0; dy < CH; ++dy)
#pragma unroll
                for (int dx = 0; dx < CW; ++dx)
#pragma unroll
                    for (int u = 0; u < 8; ++u) t[dy * CW + dx][u] = win[roff[u] + dy * g.wo + dx];
#pragma unroll
            for (int w9 = 0; w9 < CH * CW; ++w9)
#pragma unroll
                for (int u = 0; u < 8; ++u) mx[u] = __builtin_fmaxf(mx[u], t[w9][u]);
        } else {
            for (int dy = 0; dy < pp.ph; ++dy)
                for (int dx = 0; dx < pp.pw; ++dx) {
                    float t[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) t[u] = win[roff[u] + dy * g.wo + dx];
#pragma unroll
                    for (int u = 0; u < 8; ++u) mx[u] = __builtin_fmaxf(mx[u], t[u]);
                }
        }
    };
    const int wkind = (pp.ph == 3 && pp.pw == 3) ? 3 : (pp.ph == 2 && pp.pw == 2) ? 2 : 0;
#pragma unroll
    for (int i = 0; i < FW; ++i) {
#pragma unroll
        for (int hq = 0; hq < 2; ++hq) {          // filter rows 16*hq .. 16*hq + 15 of the block
#pragma unroll
            for (int j = 0; j < PW; ++j)
#pragma unroll
                for (int v8 = 0; v8 < 8; ++v8) {
                    const int v = 8 * hq + v8;
                    float y = E::to_float(acc[i][j], v) * Km[j] * al[i][v];
                    if (pp.relu) y = y > 0.0f ? y : 0.0f;
                    ystage[(8 * (v8 >> 2) + 4 * half + (v8 & 3)) * YP + (wp * PW + j) * 32 + l32] = y;
                }
            __builtin_amdgcn_wave_barrier();
            const int row0 = f0 + (wf * FW + i) * 32 + 16 * hq;
            const int nrow = min(16, g.k_out - row0);       // staged filters that exist (wave-uniform, may be <= 0)
            for (int q = pq; q < npool; q += pstep) {
                const uint32_t py = pp.div_wpo.div_small((uint32_t)q);
                const int px = q - (int)py * pp.wpo;
                const float *win = ystage + (int)py * pp.sh * g.wo + px * pp.sw;
                float *dst = pooled + ((size_t)pool_img * g.k_out + row0 + fo) * plane + (size_t)pool_py0 * pp.wpo + q;
                for (int fb = 0; fb < nrow; fb += 8 * nf) {       // wave-uniform trip count
                    int roff[8];
                    float mx[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        roff[u] = min(fb + u * nf + fo, 15) * YP;      // clamped: always inside the wave's tile
                        mx[u] = -__builtin_inff();
                    }
                    if (wkind == 3) window_max(std::integral_constant<int, 3>{}, std::integral_constant<int, 3>{}, win, roff, mx);
                    else if (wkind == 2) window_max(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{}, win, roff, mx);
                    else window_max(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, win, roff, mx);
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (lane_on && fb + u * nf + fo < nrow) in_global(dst)[(size_t)(fb + u * nf) * plane] = mx[u];
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    } else if constexpr (!FUSE) {
#pragma unroll
    for (int i = 0; i < FW; ++i) {
        float al[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {           // rows 8q + 4*half .. +3 of the block: one 16-byte read
            const float4 a4 = *reinterpret_cast<const float4 *>(par_lds + (wf * FW + i) * 32 + 8 * q + 4 * half);
            al[4 * q] = a4.x; al[4 * q + 1] = a4.y; al[4 * q + 2] = a4.z; al[4 * q + 3] = a4.w;
        }
#pragma unroll
        for (int j = 0; j < PW; ++j) {
            store_rows(out, i, j, [&](int v) {
                return __builtin_bit_cast(uint32_t, E::to_float(acc[i][j], v) * Km[j] * al[v]);
            });
            if (dot_out) store_rows(dot_out, i, j, [&](int v) { return (uint32_t)E::to_int(acc[i][j], v); });
        }
    }
    } else {
    // Fused epilogue: the next block's BatchNorm and BinActiv on y = float(dot) * K * alpha while it
    // is still in registers.  A lane holds 16 of the 32 filter rows of a block for one pixel; the
    // other 16 sit in the lane 32 further on, so one cross-half exchange completes the sign word
    // and the |z| sum of the block.  Exchanges run for every lane (dead pixel columns carry
    // clamped data); only the stores are predicated.
    const int cwn = g.fblocks;                    // words per pixel of the next layer's input
    constexpr int WT = FT / 32;                   // words per pixel this workgroup produces
    float asum[PW];
#pragma unroll
    for (int j = 0; j < PW; ++j) asum[j] = 0.0f;
#pragma unroll
    for (int i = 0; i < FW; ++i) {
        const int fblk = f0 / 32 + wf * FW + i;
        const int kb = fblk * 32 + 4 * half;
        float al[16], bs[16], bb[16];
        const bool whole = kb + 28 < g.k_out;     // all 16 rows of this lane exist (uniform per half-wave pair)
#pragma unroll
        for (int q = 0; q < 4; ++q) {           // rows 8q + 4*half .. +3 of the block: one 16-byte read each
            const int t = (wf * FW + i) * 32 + 8 * q + 4 * half;
            const float4 a4 = *reinterpret_cast<const float4 *>(par_lds + t);
            const float4 s4 = *reinterpret_cast<const float4 *>(par_lds + FT + t);
            const float4 b4 = *reinterpret_cast<const float4 *>(par_lds + 2 * FT + t);
            al[4 * q] = a4.x; al[4 * q + 1] = a4.y; al[4 * q + 2] = a4.z; al[4 * q + 3] = a4.w;
            bs[4 * q] = s4.x; bs[4 * q + 1] = s4.y; bs[4 * q + 2] = s4.z; bs[4 * q + 3] = s4.w;
            bb[4 * q] = b4.x; bb[4 * q + 1] = b4.y; bb[4 * q + 2] = b4.z; bb[4 * q + 3] = b4.w;
        }
#pragma unroll
        for (int j = 0; j < PW; ++j) {
            // sign word built at the rows' positions for half 0 (compile-time masks), moved to this
            // half's rows by one shift at the end
            uint32_t word = 0;
            float sabs = 0.0f;
            if (whole) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float y = E::to_float(acc[i][j], v) * Km[j] * al[v];
                    const float z = fmaf(y, bs[v], bb[v]);          // scale 1, shift 0 without normalisation: z == y
                    word |= z >= 0.0f ? 1u << (8 * (v >> 2) + (v & 3)) : 0u;
                    sabs += fabsf(z);
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int kr = 8 * (v >> 2) + (v & 3);
                    const bool fin = kb + kr < g.k_out;             // rows past the last filter: bit 0, no |z|
                    const float y = E::to_float(acc[i][j], v) * Km[j] * al[v];
                    const float z = fmaf(y, bs[v], bb[v]);          // scale 1, shift 0 without normalisation: z == y
                    word |= (fin && z >= 0.0f) ? 1u << kr : 0u;
                    sabs += fin ? fabsf(z) : 0.0f;
                }
            }
            word <<= 4 * half;
            if (out)                              // callers that also want the real tensor
                store_rows(out, i, j, [&](int v) {
                    return __builtin_bit_cast(uint32_t, E::to_float(acc[i][j], v) * Km[j] * al[v]);
                });
            word |= (uint32_t)__shfl_xor((int)word, 32);
            asum[j] += sabs + __shfl_xor(sabs, 32);
            if (half == 0) wtile_lds[((wp * PW + j) * 32 + l32) * WT + wf * FW + i] = word;
        }
        __builtin_amdgcn_sched_barrier(0);        // one block's alpha / scale / shift live at a time
    }
    // |z| summed over this workgroup's filters: waves along the filter axis combine through LDS in
    // a fixed order.  Sign words leave through LDS too, so that consecutive threads write
    // consecutive words of a pixel (the whole tile is one contiguous run when the workgroup holds
    // every filter).
    if (half == 0) {
#pragma unroll
        for (int j = 0; j < PW; ++j) asum_lds[wf * PT + (wp * PW + j) * 32 + l32] = asum[j];
    }
    __syncthreads();
    for (int t = tid; t < PT * WT; t += NT) {
        const uint32_t m = m0 + (uint32_t)(t / WT);
        const int fblk = f0 / 32 + t % WT;
        if (m < (uint32_t)g.m_total && fblk < cwn) in_global(fz.xbits_next)[(size_t)m * cwn + fblk] = wtile_lds[t];
    }
    for (int t = tid; t < PT; t += NT) {
        const uint32_t m = m0 + (uint32_t)t;
        if (m >= (uint32_t)g.m_total) continue;
        float sum = 0.0f;
#pragma unroll
        for (int q = 0; q < WF; ++q) sum += asum_lds[q * PT + t];
        if (pl.ftiles == 1) in_global(fz.A_next)[m] = sum / (float)g.k_out;
        else in_global(fz.workspace)[(size_t)ftile * g.m_total + m] = sum;
    }
    }
    }
}

constexpr int LDS_LIMIT = 160 * 1024;

// fuse_rows: rows of PT words for the fused epilogue's |z| sums and sign words (0 without it)
// par_bytes: alpha (fused epilogue: also scale and shift) of the workgroup's filters
// channel words per K-step and bytes of the widening table of an operand format (Enc<fmt>::BPS, LUT_BYTES)
static constexpr int fmt_bps(int fmt) { return fmt == 1 || fmt == 2 || fmt == 5 ? 2 : fmt == 4 || fmt == 6 ? 3 : 1; }
static constexpr int fmt_lut_bytes(int fmt) { return fmt == 0 ? 512 * 8 : 0; }     // int8 operands only
static size_t plan_lds_bytes(const MfmaPlan &pl, int fmt, int wp, int PT, int fuse_rows, int par_bytes)
{
    const size_t rest = (size_t)pl.region_bytes + (size_t)pl.max_rows * 4 +
                        (size_t)((pl.nsteps + KLOOP_TABLE_PAD) * fmt_bps(fmt)) * 4 + (size_t)pl.max_rows * wp * 4 +
                        (size_t)PT * 4 * (1 + fuse_rows) + 16;
    return (rest + 15) / 16 * 16 + fmt_lut_bytes(fmt) + par_bytes;       // + the widening table
}
static int plan_lut_offset(const MfmaPlan &pl, int fmt, int wp, int PT, int fuse_rows, int par_bytes)
{
    return (int)(plan_lds_bytes(pl, fmt, wp, PT, fuse_rows, par_bytes) - fmt_lut_bytes(fmt) - par_bytes);
}

static bool make_plan(const ConvGeom &g, int PT, int fmt, int lds_budget, int fuse_rows, int par_bytes, MfmaPlan *pl,
                      int rows_override = 0, bool lone = false, int most_chunks = 0x7fffffff)
{
    const int bps = fmt_bps(fmt), bpb = fmt == 1 || fmt == 5 ? Enc<1>::BPB : fmt == 2 ? Enc<2>::BPB : 32;
    const int rows = rows_override ? rows_override : worst_region_rows(g, PT, PT);
    for (int ccw = g.cw; ccw >= 1; --ccw) {
        // (packed words and digits: the last chunk may lack one word, staged as zeros)
        if (fmt == 1 || fmt == 2 ? (g.cw + ccw - 1) / ccw * ccw > g.cw + 1 : g.cw % ccw != 0) continue;
        // packed words and digits take two channel words per step: chunks must keep the words of a step together (a single word of
        // stored digits: two taps per step)
        if (ccw != g.cw && (ccw % bps) && !(g.stored_digits && ccw == 1)) continue;
        const long long row_bytes = (long long)ccw * bpb;
        const long long ps = row_bytes + ((row_bytes / 16) % 2 == 0 ? 16 : 0);
        // LDS row pitch: at least wp pixels, padded so that stepping from the last output pixel of a row
        // to the first of the next continues the bank pattern of the steps within a row
        // (sh * pitch = wo * sw * ps modulo the 256-byte bank period): operand reads of a wave that
        // spans a row boundary then stay conflict-free
        long long pitch = (long long)g.wp * ps;
        for (int add = 0; add < 256; add += 16)
            if (((long long)g.sh * (pitch + add) - (long long)g.wo * g.sw * ps) % 256 == 0) { pitch += add; break; }
        const long long region = (long long)rows * pitch;
        pl->row_pitch = (int)pitch;
        pl->cc_words = ccw;
        pl->ps = (int)ps;
        pl->max_rows = rows;
        pl->nsteps = (g.taps * ccw + bps - 1) / bps;
        pl->tap_jump = (ccw == g.cw) ? 0 : fmt == 2 && ccw == 1 ? 2 * g.cw - 2 : (g.cw - ccw) / (fmt == 1 || fmt == 2 ? 1 : bps);
        if (region >= (1ll << 30)) continue;
        pl->region_bytes = (int)region;
        const long long total = (long long)plan_lds_bytes(*pl, fmt, g.wp, PT, fuse_rows, par_bytes);
        const bool last = ccw <= bps;
        // one chunk with all channel words keeps the weight records consecutive (the K loop without
        // bookkeeping) and saves the refills: worth up to half the CU's LDS (two workgroups per CU)
        // (`lone`: the launch has at most one workgroup per CU, which may then take nearly all of the CU's LDS)
        const long long whole = lone ? 156 * 1024 : 80 * 1024;
        const long long budget = ccw == g.cw ? (lds_budget > whole ? lds_budget : whole) : lds_budget;
        if (total > budget && !last) continue;
        if (total > LDS_LIMIT && g.stored_digits && ccw > 1) continue;
        if (total > LDS_LIMIT) return false;
        MfmaPlan one;
        if ((g.cw + ccw - 1) / ccw > most_chunks &&
            make_plan(g, PT, fmt, lds_budget, fuse_rows, par_bytes, &one, rows_override, true) && one.cc_words == g.cw) {
            *pl = one;
            return true;
        }
        pl->div_wp = FastDiv::make((uint32_t)g.wp);
        pl->div_hp = FastDiv::make((uint32_t)g.hp);
        pl->div_ccw = FastDiv::make((uint32_t)ccw);
        return true;
    }
    return false;
}

// Raises a kernel's dynamic LDS limit once per instantiation (the library drives one GPU per process).  Concurrent first calls may both
// set the attribute (the call is idempotent); the flag only ever goes from false to true.
template <class Kern> static xnor_status allow_full_lds(Kern kern, std::atomic<bool> &done)
{
    if (done.load(std::memory_order_acquire)) return XNOR_OK;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            LDS_LIMIT) != hipSuccess)
        return XNOR_ERR_HIP;
    done.store(true, std::memory_order_release);
    return XNOR_OK;
}

template <int FMT, int FW, int PW, int WF, int WP, bool FUSE, int KS = 1>
static xnor_status launch_cfg(const uint32_t *xbits, const void *wimg, const float *K, const float *A,
                              const float *alpha, float *out, int32_t *dot_out, const ConvGeom &g,
                              hipStream_t stream, const FuseArgs *fz, bool strict = false)
{
    constexpr int FT = 32 * FW * WF, PT = 32 * PW * WP;
    // results are stored through a buffer resource with 32-bit offsets from the tile's first image
    const long long howo = (long long)g.ho * g.wo;
    if ((PT / howo + 2) * g.k_out * howo * 4 >= 0x7ffffff0LL) return XNOR_ERR_UNSUPPORTED;
    MfmaPlan pl;
    constexpr int FROWS = FUSE ? WF + FT / 32 : 0, PARB = (FUSE ? 3 : 1) * FT * 4;
    const long long wg_count = (long long)((g.m_total + PT - 1) / PT) * ((g.k_out + FT - 1) / FT);
    const int budget = std::max(mfma_lds_budget(), FMT == 2 && FW * PW > 6 ? 150 * 1024 : 0);      // (one workgroup per CU)
    // 4-bit operands, tiles of 16 result blocks and more: three chunks and more (two words each, as a count that has no
    // larger even divisor gives) cost more than holding every word with one workgroup per CU: 85 images of 320x31x31, 3x3
    // stride 2 -> 320, five chunks 30.4 us, whole 28.6.  (64 x 128, eight blocks: 34.5 and 39.5)
    if (!make_plan(g, PT, FMT, budget, FROWS, PARB, &pl, 0, wg_count <= 256, FMT == 1 && FW * PW * WF * WP >= 16 ? 2 : 0x7fffffff))
        return XNOR_ERR_UNSUPPORTED;
    // strict: packed words only in one chunk (the caller has another tile for the others), digits of parts only where they are ahead
    if (FMT != 2 && strict && pl.cc_words != g.cw) return XNOR_ERR_UNSUPPORTED;
    const size_t lds = plan_lds_bytes(pl, FMT, g.wp, PT, FROWS, PARB);
    if (FMT == 2 && strict) {
        // With one workgroup on a CU that has several to run nothing hides the conversion: a word's digits have to save 24 matrix
        // instructions per 32 x 32 results over their taps (a 512-filter tile holds the CU whatever it stages).  Where the words
        // come in chunks they have to save 84, or the tile one per staged word.  Parts against digits, us (saved per word): 2 images of 35x50x50, 3x3 -> 448 (18) 13.4 / 20.7;
        // 18 of 64x50x50, 3x3 -> 236 (31) 37.2 / 32.9; 88 of 32x18x43, 5x5 -> 32 (25) 35.9 / 25.3; in chunks 7 of 68x44x44, 3x3 -> 288
        // (15) 26.7 / 45.3; 5 of 160x51x51, 5x5 -> 60 (75) 49.1 / 61.4; 20 of 192x34x34, 5x5 -> 32 (87) 82.3 / 73.6;
        // 64 of 96x27x27, 5x5 -> 256 (67, 5.5 per staged word) 117 / 92.  512 filters: 19 of 37x30x30, 3x3 -> 428 (18) 25.9 / 33.9; 5 of 96x48x48, 3x3 -> 448 (24) 31.9 / 24.8.
        const bool wide = FW * PW > 6, chunks = !wide && pl.cc_words != g.cw;
        const long long saved = bwn_digits_save(g), staged = (long long)pl.max_rows * g.wp * g.cw;
        const bool ahead = chunks ? saved >= 84LL * g.cw || saved * std::min(FT / 32, g.fblocks) * (PT / 32) >= staged
                                  : saved >= 24LL * g.cw;
        if ((wide || (lds > 80 * 1024 && wg_count > 256)) && !ahead) return XNOR_ERR_UNSUPPORTED;
    }
    pl.lut_offset = plan_lut_offset(pl, FMT, g.wp, PT, FROWS, PARB);
    // two builds of every tiling: weight records consecutive (one chunk holds all channel words) or not; 4-bit operands: a
    // third, chunks staged directly
    // (a chunk of a 1x1 filter is a run of consecutive records too)
    set_direct_staging(&pl, g, FMT, PT);
    const bool linear = FMT > 1 ? pl.tap_jump == 0 || g.taps == 1 : pl.vec > 0 && pl.cc_words == g.cw;
    // waves along K: consecutive weight records only, and the partial sums need the activation region's room
    if (KS > 1 && (!linear || (size_t)pl.region_bytes < (size_t)(KS - 1) * WF * WP * FW * PW * 16 * 64 * 4))
        return XNOR_ERR_UNSUPPORTED;
    const bool direct_chunks = FMT == 1 && !linear && pl.vec > 0;
    // (parts made of digits: where all of a pixel's fitted, a word of its digits would)
    auto kern = linear          ? conv_mfma_kernel<FMT, FW, PW, WF, WP, FUSE, FMT != 6, false, KS>
                : direct_chunks ? conv_mfma_kernel<FMT, FW, PW, WF, WP, FUSE, KS != 1, false, KS, FMT == 1 && KS == 1>
                                : conv_mfma_kernel<FMT, FW, PW, WF, WP, FUSE, KS != 1, false, KS>;
    static std::atomic<bool> attr_done[3];       // per instantiation (zero-initialised: false)
    if (xnor_status s = allow_full_lds(kern, attr_done[linear ? 1 : direct_chunks ? 2 : 0])) return s;
    pl.ptiles = (g.m_total + PT - 1) / PT;
    pl.ftiles = (g.k_out + FT - 1) / FT;
    // (measured on whole benchmark steps: 64 MiB 382 us, 40 MiB 403 us, 120 MiB 408 us, never 428 us)
    // (only where the rows of 32 pixels that a wave stores cover whole 64-byte pieces: a non-temporal store of part of one is
    // not merged with its neighbour's.  200 images of 27 x 27, 64 -> 256 channels, 142 MiB: 105 us with the hint, 32 without;
    // 256 images of 14 x 14, 128 -> 512: 77 and 32; 100 of 55 x 55, 128 -> 96: 72 and 40; 28 x 28 and 56 x 56 keep it)
    pl.stream_out = (long long)g.m_total * g.k_out * 4 > (64ll << 20) && howo % 16 == 0;
    // weight-heavy: the weight image outweighs the packed activations and there are filter tiles to spread
    pl.wmajor = pl.ftiles >= 8 && (long long)g.k_out * g.taps * g.c > 4LL * g.n * g.h * g.w * g.c;
    dim3 grid((unsigned)pl.ptiles, (unsigned)pl.ftiles), block(64 * WF * WP * KS);
    if (pl.wmajor) {
        const long long wg = (long long)((pl.ftiles + 7) / 8) * pl.ptiles * 8;
        if (wg > 0x7fffffffLL) return XNOR_ERR_UNSUPPORTED;
        grid = dim3((unsigned)wg, 1u);
    }
    if (grid.y > 65535u) return XNOR_ERR_UNSUPPORTED;
    const size_t img_bytes = FMT == 1 || FMT == 2 ? wimg_pop_bytes(g.k_out, g.c, g.taps)
                             : FMT == 4 || FMT == 6 ? wimg_bf16_bytes(g.k_out, g.cw / 3, g.taps)
                             : FMT == 5 ? wimg_f4_bytes(g.k_out, g.c, g.taps)
                                        : wimg_i8_bytes(g.k_out, g.c, g.taps);
    if (img_bytes > 0x7fffffffull) return XNOR_ERR_UNSUPPORTED;
    kern<<<grid, block, lds, stream>>>(ConvArgs{xbits, reinterpret_cast<const v4i *>(wimg), K, A, alpha, out, dot_out,
                                                (uint32_t)img_bytes, g, pl, FUSE ? *fz : FuseArgs{}});
    if (xnor_status s = hip_status(hipGetLastError())) return s;
    if (FUSE && pl.ftiles > 1) {
        return launch_sum_planes(fz->workspace, fz->A_next, g.m_total, pl.ftiles, (float)g.k_out, stream);
    }
    return XNOR_OK;
}

template <int FMT>
xnor_status launch_fmt(const uint32_t *xbits, const void *wimg, const float *K, const float *A,
                              const float *alpha, float *out, int32_t *dot_out, const ConvGeom &g,
                              hipStream_t stream, const FuseArgs *fz, bool last)
{
    int tile = FMT == 6 ? 0 : mfma_tile_override(), stead = 0;      // stead: the tile that a rule for smaller launches has replaced
    if (tile == 0) {
        // Measured rules (fp4, all benchmark layers).  Up to 64 filters: 64 x 256 when that still gives every
        // CU two workgroups, else 64 x 128; up to 128 filters: 128 x 64, else 64 x 128 (fused epilogue:
        // 64 x 256 or 128 x 128, so that one workgroup holds every filter).  129..256 filters: a tile that
        // holds every filter (weights stream through L1 once per pixel tile, the fused epilogue needs no
        // partial sums), 256 x 96 or 256 x 128, whichever leaves fewer CUs idle in its last round of
        // workgroups; 4-bit operands 256 x 64 in place of 256 x 96 where that idles no more of them (three workgroups per
        // CU instead of two: 96 x 27 x 27 batch 64 20.4 -> 19.9 us).  More filters: 256 x 128 when the filter count is a
        // multiple of 256, else 128 x 128; fused epilogue with 4-bit operands up to 512 filters: 384 x 96 or 512 x 64, so
        // that one workgroup holds every filter and no second launch adds partial sums (512 filters on 7 x 7, batch 256: 22.1 -> 18.3),
        // 384 in twelve waves of 32, three per SIMD (in six of 64 two SIMDs had twice the work of the others: 128 images of 13 x 13, 256
        // channels 17.6 -> 15.2 us, 384 channels 20.0 -> 17.3; 250 images 37 -> 33; 140 of 200x13x13, 3x3 -> 300 15.4 -> 12.9).
        // Problems with few output tiles (fully connected layers: few "pixels", long K) take the largest
        // smaller tile that still gives every CU a workgroup.
        auto wgs = [&](int ft, int pt) {
            return (long long)((g.m_total + pt - 1) / pt) * ((g.k_out + ft - 1) / ft);
        };
        const int cus = 256;
        auto waste = [&](long long w) { return (double)((w + cus - 1) / cus * cus) / (double)w; };
        if (FMT == 6) tile = g.k_out <= 64 ? 2 : 1;
        else if (FMT == 2 || FMT == 4) {
            // real activations (bfloat16 parts): the K loop is 24 times longer per channel, so the
            // tiles with the larger register blocks win wherever the filter count fills them
            // (measured): up to 64 filters 64 x 256, up to 128 filters 128 x 128; beyond that the tile
            // among 256 x 96 (when one tile holds every filter), 128 x 128 and 128 x 64 that leaves the
            // fewest CUs idle in the last round, the larger one on a tie
            // (digits, 385 to 512 filters: 512 x 64, so that several words of parts are converted once: 512 x 7 x 7, batch 256, 115 -> 99 us.
            // Digits as the split wrote them, or of a single word of parts: 512 x 64, whose waves read every staged digit for four filter blocks,
            // or 256 x 96, whichever has less to do on the CU that does most (8 and 6 blocks per wave and workgroup): 256 of 512x7x7, 3x3 -> 512
            // 73 / 98 us, 64 of 256x14x14, 1x1 -> 400 16.2 / 18.1; 28 of 192x12x50, 3x3 -> 416 69 / 60, 5 of 96x48x48, 3x3 -> 448 21.7 / 18.5; one
            // word, 3 of 26x52x52, 5x5 -> 415 26.1 / 21.0, 11 of 30x30x30, 5x5 -> 385 24.7 / 21.2)
            if (g.k_out <= 64) tile = 2;
            else if (g.k_out <= 128) tile = 1;
            else if (FMT == 2 && g.k_out > 384 && g.k_out <= 512)
                tile = (!g.stored_digits && g.cw > 1) || (wgs(512, 64) + cus - 1) / cus * 8 <= (wgs(256, 96) + cus - 1) / cus * 6 ? 12 : 4;
            else {
                const double w4 = g.k_out <= 256 ? waste(wgs(256, 96)) : 1e30;
                const double w1 = waste(wgs(128, 128)), w13 = waste(wgs(128, 64));
                tile = w4 <= 1.03 * w1 && w4 <= 1.03 * w13 ? 4 : w1 <= 1.03 * w13 ? 1 : 13;
            }
        } else if (g.k_out <= 64) tile = (fz || wgs(64, 256) >= 2 * cus) ? 2 : 11;
        else if (g.k_out <= 128) tile = fz ? 1 : wgs(128, 64) >= 2 * cus ? 13 : 11;
        else if (g.k_out <= 256) {
            tile = waste(wgs(256, 96)) <= waste(wgs(256, 128)) ? 4 : 5;
            // fused epilogue, at most one workgroup per CU: eight waves of 32 filters in place of four of 64, so that a SIMD has two to
            // choose from (128 of 384x13x13, 3x3 -> 256 15.2 -> 13.7 us, 100 of 256x14x14, 3x3 -> 256 12.8 -> 11.4, 110 of 300x13x13, 1x1 ->
            // 130 9.5 -> 7.9; with several workgroups per CU the wider waves are ahead: 128 of 96x27x27, 5x5 -> 256 33 / 42)
            if (FMT == 1 && fz && wgs(256, 96) <= cus) { tile = 3; stead = 4; }
            else if (FMT == 1 && tile == 4 && waste(wgs(256, 64)) <= waste(wgs(256, 96))) { tile = 6; stead = 4; }
        } else if (FMT == 1 && fz && g.k_out <= 512) tile = g.k_out <= 384 ? 9 : 8;
        else tile = g.k_out % 256 == 0 ? 5 : fz ? 13 : 1;      // (fused epilogue: 128 x 64 ahead of 128 x 128)
        // 4-bit operands: less than a workgroup per CU of 128 x 128, 128 x 64 is ahead of it (3 images of 352x48x48 -> 310 14.6 -> 13.4 us,
        // 8 of 416x28x28 -> 390 15.8 -> 14.2, 36 of 64x14x14 -> 384 8.1 -> 7.6, 9 of 192x28x28 -> 300 1x1 7.4 -> 6.8), but for those
        // that hold every channel word with one workgroup per CU and would take chunks with two (11 images of 480x29x29, 5x5 -> 300
        // 25.6 and 36.9; 2 of 362x53x53 -> 416 13.7 and 17.6: below)
        if (FMT == 1 && tile == 1 && !fz && g.k_out > 256 && wgs(128, 128) < cus) { tile = 13; stead = 1; }
        const long long w0 = tile == 11 ? wgs(64, 128) : tile == 2 ? wgs(64, 256) : tile == 4 || tile == 3 ? wgs(256, 96)
                             : tile == 5 ? wgs(256, 128) : tile == 6 ? wgs(256, 64) : tile == 8 ? wgs(512, 64)
                             : tile == 9 ? wgs(384, 96) : tile == 12 ? wgs(512, 64) : tile == 13 ? wgs(128, 64) : wgs(128, 128);
        // (fused tiles of eight waves and more, which hold every filter: 90 of 256x13x13, 3x3 -> 320, 159 workgroups, 13.8 us, in 128 x 64 15.9)
        if (w0 < (FMT == 2 || FMT == 4 || FMT == 6 || tile == 3 || tile == 8 || tile == 9 ? 128 : 160)) {
            if (FMT == 6) tile = 14;
            else if (wgs(64, 128) >= cus) tile = 11;
            else if (wgs(128, 64) >= cus) tile = 13;
            else tile = (FMT < 2 && !fz && g.taps == 1) ? 15 : 14;       // 128 x 32 (measured ahead of 64 x 64 at equal workgroup count), with eight waves where the records are consecutive
        }
        // Fused epilogue, 129 to 512 filters, few pixels: tiles of 32 pixels whose eight or sixteen waves hold every filter save the second
        // launch that adds partial sums (2.5 us), while their waves share the SIMDs for a K loop that is not longer than that (graphs of
        // one kernel, against the best of the other tiles): 1 of 64x6x6, 3x3 -> 200 4.9 / 6.5 us, 40 of 128x14x14, 3x3 -> 200 5.9 / 8.4, 20 of
        // 256x14x14, 3x3 -> 256 7.1 / 8.7, 76 of 300x14x14, 1x1 -> 256 6.8 / 8.0; 2 of 480x14x14, 5x5 -> 160 (188 steps) 16.8 / 15.2; more than two
        // workgroups per CU, 100 of 128x14x14 -> 200 9.9 / 8.5.  Sixteen waves: 40 of 100x12x12, 1x1 -> 300 6.3 / 7.7, 3 of 200x9x9, 1x1 -> 400
        // 6.3 / 7.0, 10 of 96x8x8, 3x3 -> 384 (27 steps) 7.2 / 7.2, 1 of 300x6x6, 5x5 -> 500 18.0 / 11.7; 51 of 256x14x14, 1x1 -> 400, 313
        // workgroups, 11.1 / 8.0.
        const int steps = (g.taps * g.cw + 1) / 2;
        if (FMT == 1 && fz && g.k_out > 128) {
            const int small = g.k_out <= 256 && wgs(256, 32) <= 2 * cus && steps <= 150 ? 7
                              : g.k_out > 256 && g.k_out <= 512 && wgs(512, 32) <= cus && steps <= 24 ? 10 : 0;
            if (small) { stead = stead ? stead : tile; tile = small; }
        }
    }
    // every tiling is built with and without the fused epilogue (bfloat16 parts and k-bit levels: without only)
#define XNOR_TILE_F(ID, FW, PW, WF, WP)                                                                   \
    case ID:                                                                                              \
        if constexpr (FMT == 6 && ID != 1 && ID != 2 && ID != 14) return XNOR_ERR_UNSUPPORTED;            \
        else {                                                                                            \
        if constexpr (FMT < 2) {                                                                          \
            if (fz) return launch_cfg<FMT, FW, PW, WF, WP, true>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, fz); \
        }                                                                                                 \
        return launch_cfg<FMT, FW, PW, WF, WP, false>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, nullptr, strict); }
#define XNOR_TILE_F4(ID, FW, PW, WF, WP)                                                                  \
    case ID:                                                                                              \
        if constexpr (FMT == 1)                                                                           \
            return fz ? launch_cfg<FMT, FW, PW, WF, WP, true>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, fz)        \
                      : launch_cfg<FMT, FW, PW, WF, WP, false>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, nullptr); \
        return XNOR_ERR_UNSUPPORTED;
    auto launch = [&](int tile, bool strict = false) -> xnor_status {
    switch (tile) {
        XNOR_TILE_F(1, 2, 2, 2, 2);   // 128 filters x 128 pixels
        XNOR_TILE_F(2, 2, 2, 1, 4);   //  64 x 256
        XNOR_TILE_F(4, 2, 3, 4, 1);   // 256 x  96
        XNOR_TILE_F(5, 2, 4, 4, 1);   // 256 x 128
        XNOR_TILE_F4(6, 2, 2, 4, 1);  // 256 x  64
        XNOR_TILE_F(11, 1, 2, 2, 2);  //  64 x 128
        XNOR_TILE_F(13, 1, 2, 4, 1);  // 128 x  64
        XNOR_TILE_F(14, 1, 1, 4, 1);  // 128 x  32
    case 12:                          // 512 x  64, one workgroup of four waves per CU (digit operands)
        if constexpr (FMT == 2) return launch_cfg<FMT, 4, 2, 4, 1, false>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, nullptr, strict);
        return XNOR_ERR_UNSUPPORTED;
    case 7:                           // 256 x  32, eight waves,
    case 10:                          // 512 x  32, sixteen,
    case 3:                           // 256 x  96, eight,
    case 8:                           // 512 x  64, eight, and
    case 9:                           // 384 x  96, twelve: one workgroup holds every filter of the fused epilogue (4-bit operands)
        if constexpr (FMT == 1) {
            if (fz && tile == 7) return launch_cfg<FMT, 1, 1, 8, 1, true>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, fz);
            if (fz && tile == 10) return launch_cfg<FMT, 1, 1, 16, 1, true>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, fz);
            if (fz && tile == 3) return launch_cfg<FMT, 1, 3, 8, 1, true>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, fz);
            if (fz && tile == 8) return launch_cfg<FMT, 2, 2, 8, 1, true>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, fz);
            if (fz) return launch_cfg<FMT, 1, 3, 12, 1, true>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, fz);
        }
        return XNOR_ERR_UNSUPPORTED;
    case 15:                          // 128 x  32, two groups of four waves along K (no fused epilogue, packed-bit operands)
        if constexpr (FMT < 2) {
            if (!fz) {
                const xnor_status s = launch_cfg<FMT, 1, 1, 4, 1, false, 2>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, nullptr);
                // (the library's own choice falls back to the four-wave form where this one does not apply)
                if (s != XNOR_ERR_UNSUPPORTED || mfma_tile_override() == 15) return s;
                return launch_cfg<FMT, 1, 1, 4, 1, false>(xbits, wimg, K, A, alpha, out, dot_out, g, stream, nullptr);
            }
        }
        return XNOR_ERR_UNSUPPORTED;
    default: return XNOR_ERR_UNSUPPORTED;
    }
    };
#undef XNOR_TILE_F
#undef XNOR_TILE_F4
    xnor_status s = launch(tile, FMT == 2 ? !last && mfma_tile_override() == 0 : stead == 1);
    if (stead == 1 && s == XNOR_ERR_UNSUPPORTED) s = launch(1, true);
    if (stead == 1 && s == XNOR_ERR_UNSUPPORTED) s = launch(13);
    // Real inputs, many rows under a tile: fewer pixels span fewer of them.  (Parts, where nothing else takes the call: 32 pixels fit wherever
    // any tile does)
    if (FMT == 2 && tile == 4 && !g.stored_digits && g.k_out > 384 && mfma_tile_override() == 0 && s == XNOR_ERR_UNSUPPORTED) s = launch(12);
    if (FMT == 2 && g.stored_digits && mfma_tile_override() == 0)
        for (const int other : {11, 14})
            if (s == XNOR_ERR_UNSUPPORTED) s = launch(other);
    if ((FMT == 6 || (FMT == 4 && last && mfma_tile_override() == 0)) && tile != 14 && s == XNOR_ERR_UNSUPPORTED) s = launch(14);
    if (FMT != 1 || mfma_tile_override() != 0) return s;
    // 4-bit operands: the rows under the chosen tile may not fit the LDS with what the tile keeps beside them (384 and 512
    // filters of the fused epilogue: 5 and 6 KiB of alpha, scale and shift, a word per pixel and 32 filters; 64 x 6 x 6, one 6 x 6
    // window, fused with 384 filters: 190 KB for 384 x 96, 123 KB for 128 x 64).  Where nothing else takes the call, fewer
    // pixels and filters do.  Where the vector ALU does, it stays ahead of them as often as not (7 x 40 x 804, 7 x 7 -> 300,
    // 24 images: 893 us against 3215; 160 x 21 x 119, 11 x 11 stride 2 -> 512, 19 images: 362 against 206).
    for (const int other : {stead, last ? 13 : 0, last ? 14 : 0})
        if (s == XNOR_ERR_UNSUPPORTED && other) s = launch(other);
    return s;
}

}  // namespace xnor
