// BinActiv layer (sec. 3.2): sign(I) packed to bits, A = channel mean of |I|, K = box filter of A.
// Optional batch normalisation folded in front (block order BatchNorm -> BinActiv).
#include "xnor_internal.h"
#include <atomic>
#include <algorithm>

namespace xnor {

// One workgroup = up to 64 pixels that follow each other in an image x all channels (small planes: in the batch, launch_binactiv).  Lanes run
// along the pixels (contiguous in NCHW, so every channel row is read as 256-byte coalesced segments); the NW waves
// share the channels in groups of 8 (wave w takes groups w, w+NW, ...), so any channel count keeps
// all waves busy with many independent loads in flight.  A group's 8 sign bits are one byte of
// the pixel's packed word: it is assembled in LDS, from where the words of the tile leave
// as one contiguous, fully coalesced run.  |y| is accumulated per wave in float; the NW partial
// sums per pixel meet in LDS in a fixed order, so results do not depend on timing.
// What bounds it: memory (256 of 64x56x56: 32.7 us, 6.3 TB/s), on small inputs the launch and one trip to memory.  Masks only in a last group that
// lacks channels, and the waves of binactiv_waves, against masks in every group and 4 or 16 waves, us in a graph: 128 of 256x13x13, normalised
// 7.1 -> 4.4, 256 of 128x28x28 18.3 -> 17.1, 256 of 512x7x7 5.1 -> 4.3, 256 of 64x56x56 34.5 -> 32.7, 9 of 83x29x23 3.2 -> 2.9.
// Max-pooling in front of the layer (block order BinConv -> Pool -> next block's BatchNorm -> BinActiv,
// sec. 3.2): `hw` then counts pooled pixels and every value is the maximum of its window of the
// h x w input plane.  Out-of-range window positions are skipped; the maximum starts at -inf and skips
// NaN inputs (maxNum), so it is never NaN itself.
struct PoolGeom {
    int h, w, wo;           // input plane, pooled row length
    int ph, pw, sh, sw;     // window, stride
    int pad_h, pad_w;
    int relu;               // max(., 0) before the normalisation (the optional ReLU of sec. 3.2)
    int stage;              // > 0: floats per channel of the per-wave LDS staging buffer (see the kernel)
    int px_tile;            // pixels per workgroup, at most 64
    int tiles;              // workgroups per image; 0 (unpooled form): the pixels of the whole batch in one row
    int streamed;           // unpooled form: the caller says the input is not in any cache (read with the non-temporal hint)
};

// NW = waves per workgroup (launch_binactiv_impl).  The pooled form runs 16: a pooled image has few pixels (13 x 13 after
// the 27 x 27 layer), so 64-pixel tiles alone would leave CUs idle and each wave with hundreds of
// dependent window loads; more waves share the channels instead.
// PH x PW > 0: pooling window known at compile time (3 x 3 and 2 x 2 are built): all window loads of
// a channel group are then in flight together; 0: any window, one window position at a time.
// STREAM: the float input is read with the non-temporal hint (see the loads).
template <bool WRITE_BITS, bool WRITE_A, bool BN, bool POOL, int NW, int PH = 0, int PW = 0, bool STREAM = false>
__global__ __launch_bounds__(64 * NW) void binactiv_kernel(
    const float *__restrict__ x, const float *__restrict__ bn_scale,
    const float *__restrict__ bn_shift, uint32_t *__restrict__ xbits, float *__restrict__ A,
    int c, int hw, int cw, int nblocks, int px_tile, uint32_t len, FastDiv div_tiles, FastDiv div_hw, PoolGeom pg)
{
    // Workgroups are dealt to the 8 XCDs round-robin by index.  Neighbouring pixel tiles share the
    // cache lines that straddle their boundary (channel rows are not line aligned), so within
    // every window of 64 tiles each XCD takes a run of 8 consecutive ones: the shared line is then
    // a hit in that XCD's own L2, while all XCDs still stream through the same region of memory.
    // The last, incomplete window keeps the plain order (runs would load the XCDs unevenly there).
    const unsigned b = blockIdx.x, win = (b >> 6) << 6;
    const int blk = (int)(win + 64u <= (unsigned)nblocks ? win + ((b & 7u) << 3) + ((b >> 3) & 7u) : b);
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    float(*part)[64] = reinterpret_cast<float(*)[64]>(smem);            // [NW][64]
    uint8_t *wbytes = smem + NW * 64 * sizeof(float);                   // [64 px][cw words][4 bytes]
    float *stage_lds = reinterpret_cast<float *>(wbytes + (size_t)64 * cw * 4);   // [NW][2][pg.stage], pooled form
    const int tid = threadIdx.x;
    // the wave index as a scalar: channel indices derived from it are then scalar too, and the
    // per-channel scale and shift come through the scalar cache instead of 64-lane loads
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // a row of `tiles` tiles over `len` pixels: an image, or (unpooled form, planes of less than 64 pixels) the whole batch
    const uint32_t row = div_tiles.div((uint32_t)blk);
    const uint32_t p0 = ((uint32_t)blk - row * div_tiles.d) * (uint32_t)px_tile, first = row * len + p0;
    const int npx = (int)min((uint32_t)px_tile, len - p0);
    const bool live = lane < npx;
    const uint32_t m = first + (uint32_t)min(lane, npx - 1);              // of the batch
    const uint32_t img_l = POOL ? row : div_hw.div(m);
    const float *xi = x + (size_t)img_l * c * hw + (m - img_l * (uint32_t)hw);      // unpooled: this lane's pixel
    const int img = (int)row, pc = (int)(m - row * len);                  // pooled: the image, this lane's pixel there
    const float *xs = x + (size_t)img * c * pg.h * pg.w;                  // pooled: the image (wave-uniform)
    const int in_hw = POOL ? pg.h * pg.w : hw;
    int iy0 = 0, ix0 = 0;       // window origin of this lane's pooled pixel
    if (POOL) {
        const int oy = pc / pg.wo;
        iy0 = oy * pg.sh - pg.pad_h;
        ix0 = (pc - oy * pg.wo) * pg.sw - pg.pad_w;
    }
    const int groups = (c + 7) >> 3;
    float asum = 0.0f;
    // Every load is unconditional (indices clamped into the tensor) so that the 8 loads of a group,
    // and those of the next groups, are all in flight together; validity is applied afterwards.
#pragma unroll 4
    for (int gidx = wave; gidx < groups; gidx += NW) {
        const int ch0 = gidx * 8;
        float v[8];
        if (!POOL) {
            // An input beyond a quarter of the 256 MB last-level cache cannot be resident anyway and is read once: the
            // non-temporal hint keeps its stream from displacing the previous layers' results, which still wait in that
            // cache to be written back (a whole benchmark step 428 -> 412 us).  Smaller inputs keep the default policy:
            // they are often the previous layer's result, still in cache (with the hint a chain of three 13 x 13 blocks
            // took 93 instead of 86 us).
            if constexpr (STREAM) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(xi + (size_t)min(ch0 + j, c - 1) * in_hw);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = xi[(size_t)min(ch0 + j, c - 1) * in_hw];
            }
        } else if constexpr (PH > 0) {
            uint32_t off[PH * PW];       // byte offsets within the channel plane (unsigned: scalar base + 32-bit lane offset)
            bool okw[PH * PW];
#pragma unroll
            for (int dy = 0; dy < PH; ++dy)
#pragma unroll
                for (int dx = 0; dx < PW; ++dx) {
                    const int iy = iy0 + dy, ix = ix0 + dx;
                    okw[dy * PW + dx] = (unsigned)iy < (unsigned)pg.h && (unsigned)ix < (unsigned)pg.w;
                    off[dy * PW + dx] = (uint32_t)(min(max(iy, 0), pg.h - 1) * pg.w + min(max(ix, 0), pg.w - 1)) * 4u;
                }
            // maximum that skips NaN and starts at -inf (never NaN itself); positions outside the
            // image count as -inf
            const bool padded = pg.pad_h != 0 || pg.pad_w != 0;
            auto window_max = [&](const float (&t)[PH * PW]) {
                float m = -__builtin_inff();
                if (padded) {
#pragma unroll
                    for (int q = 0; q < PH * PW; ++q) m = __builtin_fmaxf(m, okw[q] ? t[q] : -__builtin_inff());
                } else {
#pragma unroll
                    for (int q = 0; q < PH * PW; ++q) m = __builtin_fmaxf(m, t[q]);
                }
                return m;
            };
            if (pg.stage > 0) {
                // The windows of neighbouring pooled pixels overlap and sit two floats apart, so loading
                // them lane by lane moves every input element several times through L1 in half-used
                // lines.  Instead the wave copies the input rows its tile touches (one contiguous run
                // per channel) into a private LDS buffer, two channels at a time, fully coalesced and
                // once, and the lanes pick their windows out of LDS.  LDS serves one wave's
                // instructions in order, so the copy needs no barrier beyond the compiler's.
                const int oy_a = p0 / pg.wo, oy_b = min(p0 + 63, hw - 1) / pg.wo;
                const int r0 = max(oy_a * pg.sh - pg.pad_h, 0);
                const int r1 = min(oy_b * pg.sh - pg.pad_h + PH - 1, pg.h - 1);
                const int nfl = (r1 - r0 + 1) * pg.w;             // <= pg.stage by the host's bound
                float *stg = stage_lds + (size_t)wave * 2 * pg.stage;
                uint32_t loff[PH * PW];
#pragma unroll
                for (int q = 0; q < PH * PW; ++q) loff[q] = off[q] / 4u - (uint32_t)(r0 * pg.w);
#pragma unroll
                for (int pr = 0; pr < 4; ++pr) {
                    float r[2][8];              // nfl <= 512 = 8 * 64: all loads of the pair in flight together
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const float *plane = xs + (size_t)min(ch0 + 2 * pr + u, c - 1) * in_hw + r0 * pg.w;
#pragma unroll
                        for (int k = 0; k < 8; ++k) r[u][k] = plane[min(lane + 64 * k, nfl - 1)];
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            if (lane + 64 * k < nfl) stg[u * pg.stage + lane + 64 * k] = r[u][k];
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        float t[PH * PW];
#pragma unroll
                        for (int q = 0; q < PH * PW; ++q) t[q] = stg[u * pg.stage + loff[q]];
                        v[2 * pr + u] = window_max(t);
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            } else {
                float tt[8][PH * PW];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const char *plane = reinterpret_cast<const char *>(xs + (size_t)min(ch0 + j, c - 1) * in_hw);
#pragma unroll
                    for (int q = 0; q < PH * PW; ++q) tt[j][q] = *reinterpret_cast<const float *>(plane + off[q]);
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = window_max(tt[j]);
            }
            if (pg.relu) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = v[j] > 0.0f ? v[j] : 0.0f;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = -__builtin_inff();
            for (int dy = 0; dy < pg.ph; ++dy) {
                const int iy = iy0 + dy;
                const bool oky = (unsigned)iy < (unsigned)pg.h;
                const int rowoff = min(max(iy, 0), pg.h - 1) * pg.w;
                for (int dx = 0; dx < pg.pw; ++dx) {
                    const int ix = ix0 + dx;
                    const bool ok = oky && (unsigned)ix < (unsigned)pg.w;
                    const int off = rowoff + min(max(ix, 0), pg.w - 1);
                    float t[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) t[j] = xs[(size_t)min(ch0 + j, c - 1) * in_hw + off];
#pragma unroll
                    for (int j = 0; j < 8; ++j) v[j] = __builtin_fmaxf(v[j], ok ? t[j] : -__builtin_inff());
                }
            }
            if (pg.relu) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = v[j] > 0.0f ? v[j] : 0.0f;     // never NaN here
            }
        }
        uint32_t byte = 0;
        auto sign_and_sum = [&](int real) {                   // channels of the group that exist
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (j >= real) break;
                const float y = BN ? __builtin_fmaf(v[j], bn_scale[ch0 + j], bn_shift[ch0 + j]) : v[j];
                byte |= y >= 0.0f ? 1u << j : 0u;
                asum += __builtin_fabsf(y);
            }
        };
        if (ch0 + 8 <= c) sign_and_sum(8);
        else sign_and_sum(c - ch0);
        if (WRITE_BITS) wbytes[(lane * cw) * 4 + gidx] = (uint8_t)byte;   // byte gidx of the pixel's word run
    }
    if (WRITE_A) part[wave][lane] = asum;
    __syncthreads();
    if (WRITE_A && wave == 0 && live) {
        float s = part[0][lane];
#pragma unroll
        for (int q = 1; q < NW; ++q) s += part[q][lane];
        A[first + lane] = s / (float)c;
    }
    if (WRITE_BITS) {
        const uint32_t *wsrc = reinterpret_cast<const uint32_t *>(wbytes);
        uint32_t *dst = xbits + (size_t)first * cw;
        const int nwords = npx * cw;
        const int tail_bytes = cw * 4 - groups;          // bytes of the last word no group wrote
        const uint32_t tail_mask = 0xFFFFFFFFu >> (8 * tail_bytes);
        int wd = tid % cw;                                // word index within the pixel, advanced by NT % cw
        const int wstep = (64 * NW) % cw;
        for (int i = tid; i < nwords; i += 64 * NW) {
            uint32_t word = wsrc[i];
            if (wd == cw - 1) word &= tail_mask;
            dst[i] = word;
            wd += wstep;
            if (wd >= cw) wd -= cw;
        }
    }
}

// hw == 1 (fully connected layers): the channels of one image are contiguous, so lanes run along
// channels and a wave-wide comparison yields 64 sign bits (two packed words) at once.  One workgroup of
// NWV waves per image (16 for long rows: a batch is a few hundred workgroups, so the loads in flight per
// CU come from the waves of one workgroup).
template <int NWV>
__global__ __launch_bounds__(64 * NWV) void binactiv_vec_kernel(
    const float *__restrict__ x, const float *__restrict__ bn_scale,
    const float *__restrict__ bn_shift, uint32_t *__restrict__ xbits, float *__restrict__ A,
    int c, int cw)
{
    __shared__ float part[NWV];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int img = blockIdx.x;
    const float *xi = x + (size_t)img * c;
    const bool bn = bn_scale != nullptr;
    float asum = 0.0f;
    // up to twelve 64-channel segments per wave and turn: the loads (clamped; segments past the last channel are skipped,
    // which is uniform per wave) are all in flight together, so a row of 9216 channels costs one trip to memory, not three
    constexpr int SEG = 12;
    for (int base0 = wave * 64; base0 < c; base0 += 64 * SEG * NWV) {
        float v[SEG], sc[SEG], sh[SEG];
#pragma unroll
        for (int u = 0; u < SEG; ++u) {
            v[u] = 0.0f; sc[u] = 1.0f; sh[u] = 0.0f;
            if (base0 + u * 64 * NWV < c) {
                const int chc = min(base0 + u * 64 * NWV + lane, c - 1);
                v[u] = xi[chc];
                if (bn) { sc[u] = bn_scale[chc]; sh[u] = bn_shift[chc]; }
            }
        }
#pragma unroll
        for (int u = 0; u < SEG; ++u) {
            const int base = base0 + u * 64 * NWV, ch = base + lane;
            const float y = bn ? __builtin_fmaf(v[u], sc[u], sh[u]) : v[u];
            const bool ok = ch < c;
            asum += ok ? __builtin_fabsf(y) : 0.0f;
            const unsigned long long mask = __ballot(ok && y >= 0.0f);
            if (xbits && base < c) {
                const int wd = base >> 5;
                if (lane == 0) xbits[(size_t)img * cw + wd] = (uint32_t)mask;
                if (lane == 1 && wd + 1 < cw) xbits[(size_t)img * cw + wd + 1] = (uint32_t)(mask >> 32);
            }
        }
    }
    if (A) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) asum += __shfl_xor(asum, off, 64);
        if (lane == 0) part[wave] = asum;
        __syncthreads();
        if (tid == 0) {
            float s = part[0];
#pragma unroll
            for (int q = 1; q < NWV; ++q) s += part[q];        // fixed order
            A[img] = s / (float)c;
        }
    }
}

template <bool WB, bool WA, bool BN, bool POOL, int NW, int PH, int PW>
static xnor_status launch_binactiv_one(dim3 grid, size_t lds, hipStream_t stream, const float *x,
                                       const float *bn_scale, const float *bn_shift, uint32_t *xbits, float *A, int n, int c,
                                       int hw, int cw, int blocks, const PoolGeom &pg)
{
    // (the cache policy is an instruction field: a kernel of its own for streamed inputs)
    const bool stream_in = !POOL && (pg.streamed || (long long)n * c * hw * 4 > (64ll << 20));
    auto kern = stream_in ? binactiv_kernel<WB, WA, BN, POOL, NW, PH, PW, !POOL> : binactiv_kernel<WB, WA, BN, POOL, NW, PH, PW, false>;
    if (lds > 48 * 1024) {      // the pooled form's staging buffer can pass the default dynamic LDS limit
        static std::atomic<bool> attr_done[2];   // per kernel; false -> true only, a repeated attribute call is harmless
        if (!attr_done[stream_in].load(std::memory_order_acquire)) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    160 * 1024) != hipSuccess)
                return XNOR_ERR_HIP;
            attr_done[stream_in].store(true, std::memory_order_release);
        }
    }
    const bool per_image = pg.tiles > 0;
    kern<<<grid, dim3(64 * NW), lds, stream>>>(x, bn_scale, bn_shift, xbits, A, c, hw, cw, blocks, pg.px_tile,
                                               per_image ? (uint32_t)hw : (uint32_t)((long long)n * hw),
                                               FastDiv::make((uint32_t)(per_image ? pg.tiles : blocks)), FastDiv::make((uint32_t)hw), pg);
    return hip_status(hipGetLastError());
}

static long long binactiv_blocks(int n, int hw, const PoolGeom &pg)
{
    return pg.tiles ? (long long)n * pg.tiles : ((long long)n * hw + pg.px_tile - 1) / pg.px_tile;
}

// LDS of a workgroup: a partial sum per wave and pixel, the words of 64 pixels
constexpr size_t BINACTIV_LDS = 64 * 1024;
static size_t binactiv_lds(int waves, int cw) { return (size_t)waves * 64 * sizeof(float) + (size_t)64 * cw * 4; }

// Waves per workgroup of the unpooled form, each at least a group of 8 channels.  A CU holds 2048 threads: 256 CUs take 2048 workgroups of four
// waves in one round, 1024 of eight, 512 of sixteen.  Few workgroups want many loads in flight each, more of them want one round.  Over 700
// layers, time against the best of the three in the mean, four / eight / sixteen waves, inputs cached and from memory:
//   8 to 15 groups, up to 256 workgroups 1.06 / 1.00 / 1.03 and 1.06 / 1.00 / 1.02, to 2048 1.00 / 1.10 / 1.25 and 1.01 / 1.01 / 1.16, more 1.02 / 1.00 / 1.41
//   16 to 23, up to 256 1.10 / 1.00 / 1.05 and 1.15 / 1.01 / 1.02, to 512 1.00 / 1.05 / 1.18 and 1.03 / 1.01 / 1.02, to 1024 1.00 / 1.08 / 1.30 and
//   1.01 / 1.00 / 1.11, more 1.02 / 1.00 / 1.18 and 1.05 / 1.00 / 1.17
//   24 to 39, up to 256 1.20 / 1.00 / 1.02 and 1.32 / 1.04 / 1.00, to 512 1.13 / 1.00 / 1.09 and 1.08 / 1.02 / 1.00, to 1024 1.01 / 1.01 / 1.06 and
//   1.01 / 1.04 / 1.06, more 1.08 / 1.01 / 1.07 and 1.08 / 1.01 / 1.06
//   40 and more, up to 256 1.37 / 1.05 / 1.00 and 1.64 / 1.14 / 1.00, to 512 1.12 / 1.01 / 1.01 and 1.22 / 1.01 / 1.03, more 1.06 / 1.07 / 1.02 and
//   1.06 / 1.08 / 1.02
static int binactiv_waves(int groups, long long blocks)
{
    if (groups < 8) return 4;
    if (blocks <= 256) return groups >= 24 ? 16 : 8;
    if (groups >= 40 && blocks > 512) return 16;
    if (groups >= 16 && blocks <= 512) return 8;
    return blocks <= (groups < 16 ? 2048 : 1024) ? 4 : 8;
}

template <bool POOL, int PH, int PW, int NW>
static xnor_status launch_binactiv_nw(const float *x, const float *bn_scale, const float *bn_shift,
                                      uint32_t *xbits, float *A, int n, int c, int hw, const PoolGeom &pg,
                                      hipStream_t stream);

template <bool POOL, int PH = 0, int PW = 0>
static xnor_status launch_binactiv_impl(const float *x, const float *bn_scale, const float *bn_shift,
                                        uint32_t *xbits, float *A, int n, int c, int hw, const PoolGeom &pg,
                                        hipStream_t stream)
{
    const long long blocks = binactiv_blocks(n, hw, pg);
    if (blocks > 0x7ffffff0LL) return XNOR_ERR_SHAPE;
    // 16 waves per workgroup for the pooled form.
    if constexpr (!POOL) {
        const int groups = (c + 7) / 8, cw = (c + 31) / 32;
        int nw = binactiv_waves(groups, blocks);
        while (nw > 4 && binactiv_lds(nw, cw) > BINACTIV_LDS) nw /= 2;         // (from 7681 channels on fewer waves leave room for the words)
        if (nw == 16) return launch_binactiv_nw<POOL, PH, PW, 16>(x, bn_scale, bn_shift, xbits, A, n, c, hw, pg, stream);
        if (nw == 8) return launch_binactiv_nw<POOL, PH, PW, 8>(x, bn_scale, bn_shift, xbits, A, n, c, hw, pg, stream);
    }
    return launch_binactiv_nw<POOL, PH, PW, POOL ? 16 : 4>(x, bn_scale, bn_shift, xbits, A, n, c, hw, pg, stream);
}

template <bool POOL, int PH, int PW, int NW>
static xnor_status launch_binactiv_nw(const float *x, const float *bn_scale, const float *bn_shift,
                                      uint32_t *xbits, float *A, int n, int c, int hw, const PoolGeom &pg,
                                      hipStream_t stream)
{
    const int cw = (c + 31) / 32;
    const long long blocks = binactiv_blocks(n, hw, pg);
    size_t lds = binactiv_lds(NW, cw);
    if (lds > BINACTIV_LDS) return XNOR_ERR_UNSUPPORTED;    // more than 8064 channels per pixel (four waves; pooled, sixteen: 7680)
    lds += (size_t)NW * 2 * pg.stage * sizeof(float);
    dim3 grid((unsigned)blocks);
#define XNOR_BA(B, AA, N) \
    return launch_binactiv_one<B, AA, N, POOL, NW, PH, PW>(grid, lds, stream, x, bn_scale, bn_shift, xbits, A, n, c, hw, cw, \
                                                           (int)blocks, pg)
    const bool bn = bn_scale != nullptr;
    if (xbits && A) { if (bn) XNOR_BA(true, true, true); else XNOR_BA(true, true, false); }
    else if (xbits) { if (bn) XNOR_BA(true, false, true); else XNOR_BA(true, false, false); }
    else            { if (bn) XNOR_BA(false, true, true); else XNOR_BA(false, true, false); }
#undef XNOR_BA
}

xnor_status launch_binactiv(const float *x, const float *bn_scale, const float *bn_shift,
                            uint32_t *xbits, float *A, int n, int c, int hw, hipStream_t stream, int streamed)
{
    if (hw == 1) {
        const int cw = (c + 31) / 32;
        if (c >= 4096)
            binactiv_vec_kernel<16><<<dim3((unsigned)n), dim3(1024), 0, stream>>>(x, bn_scale, bn_shift, xbits, A, c, cw);
        else
            binactiv_vec_kernel<4><<<dim3((unsigned)n), dim3(256), 0, stream>>>(x, bn_scale, bn_shift, xbits, A, c, cw);
        return hip_status(hipGetLastError());
    }
    PoolGeom pg{};
    pg.streamed = streamed;
    // Planes of 64 pixels and more: tiles within an image, so that a wave reads one run per channel and no cache line twice.  With the pixels of
    // the whole batch in a row a tile crosses into the next image's planes: 80 of 512x27x27 from memory 24 us / 30, 200 of 512x13x13 17 / 21, 150 of
    // 384x15x15 12.7 / 15.2, 256 of 64x56x56 (no tile crosses) 32.7 / 33.2.  Smaller planes (256 of 512x7x7 4.2 / 5.1), and batches that one
    // workgroup per CU holds only in a row (129 of 512x10x10 9.1 / 11.0, 65 of 64x15x15 3.2 / 3.4), are taken in a row.
    const long long pixels = (long long)n * hw;
    const int tiles = (hw + 63) / 64;
    if (hw >= 64 && ((long long)n * tiles <= 256 || pixels > 256 * 64)) {
        pg.tiles = tiles;
        // (a last tile of at most 8 pixels is shared out among the others: 256 of 256x14x14, tiles of 49, 11.3 us, of 64 and 4, 11.7)
        pg.px_tile = hw - (tiles - 1) * 64 <= 8 ? (hw + tiles - 1) / tiles : 64;
    } else {
        // One workgroup per CU while there are 16 pixels for each: 200 of 512x3x3 from memory, 29 workgroups of 64 pixels 8.8 us, 113 of 16 5.7 (an
        // image each 5.6); 64 of 512x5x5 6.9 and 5.2.  Whole images where that makes at least half as many: 200 of 512x7x7 from memory, 252
        // workgroups of 39 6.9, 200 of 49 6.3.  Then up to 8 per CU, the same number on each where that leaves them at least 48 pixels: 256 of 512x7x7,
        // 196 workgroups of 64 5.3 us, 256 of 49 4.05
        const long long per_cu = (pixels + 256 * 64 - 1) / (256 * 64), even = (pixels + 256 * per_cu - 1) / (256 * per_cu);
        pg.px_tile = 64;
        if (per_cu == 1) {
            pg.px_tile = (int)std::max<long long>(even, 16);
            if (hw > pg.px_tile && hw < 2 * pg.px_tile && hw <= 64) pg.px_tile = hw;
        } else if (per_cu <= 8 && even >= 48) {
            pg.px_tile = (int)even;
        }
    }
    return launch_binactiv_impl<false>(x, bn_scale, bn_shift, xbits, A, n, c, hw, pg, stream);
}

// Max-pooling of stride 2 (3 x 3 and 2 x 2 windows, rows of at most 64 pixels with their padding) in front of the layer: the same layer as
// the pooled form above, R pooled rows of an image per workgroup.  Lanes run along the columns of an input row, as many channels side by side as
// fit a wave (`lanes` = 8, 16, 32 or 64 lanes each); every lane takes 8 channels (a byte of its pixel's words), loads the rows under the R
// windows once, all of them in flight, and takes the maxima down its column in registers; two lane shifts bring in the neighbouring columns.
// Even columns then hold a pooled pixel each.  Nothing is staged, no window is read from LDS.
// What bounds it: memory, once there are workgroups and loads enough.  Against 64 pooled pixels per workgroup whose input rows went
// through LDS, two channels at a time, us: 64 of 256x27x27, 3x3 15.3 -> 11.7; 128 of 256x13x13, 3x3 12.1 -> 6.5; 256 of 128x28x28, 3x3
// 29.5 -> 18.8; 256 of 512x7x7, 2x2 18.4 -> 6.6; 256 of 256x14x14, 2x2 12.6 -> 11.3; 1 of 64x14x14, 3x3 5.9 -> 3.8; 20 of 200x56x56, 3x3
// 15.4 -> 15.2.
// Maxima start at -inf and skip NaN, as above.
__device__ __forceinline__ float next_lane(float v)      // the value of the lane above (the last lane keeps its own)
{
    const int i = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, 0x130, 0xf, 0xf, false));      // wave_shl:1
}

template <int PH, int R, int NW>
__global__ __launch_bounds__(64 * NW, NW == 16 ? 8 : 6) void pool_rows_kernel(
    const float *__restrict__ x, const float *__restrict__ bn_scale, const float *__restrict__ bn_shift,
    uint32_t *__restrict__ xbits, float *__restrict__ A, int c, int cw, int ho, int tiles_per_image, int nblocks, int lanes_log2, PoolGeom pg)
{
    constexpr int NR = 2 * (R - 1) + PH;          // input rows under the tile
    const unsigned b = blockIdx.x, win = (b >> 6) << 6;      // (runs of 8 tiles per XCD: neighbouring tiles share input rows)
    const int blk = (int)(win + 64u <= (unsigned)nblocks ? win + ((b & 7u) << 3) + ((b >> 3) & 7u) : b);
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int side = 64 >> lanes_log2;            // channel groups side by side
    const int npx = R * pg.wo;
    uint8_t *wbytes = smem;                                                            // [npx][cw words][4 bytes]
    float *part = reinterpret_cast<float *>(smem + (size_t)npx * cw * 4);              // [NW * side][npx]
    float *bn = part + NW * side * npx;                                                // scale, shift [cw * 32] each
    const int img = blk / tiles_per_image;
    const int oy0 = (blk - img * tiles_per_image) * R;
    const int rows_out = min(R, ho - oy0);
    const int col = lane & ((1 << lanes_log2) - 1), slot = wave * side + (lane >> lanes_log2);
    const int in_hw = pg.h * pg.w, xc = col - pg.pad_w;
    const bool in_row = xc >= 0 && xc < pg.w;
    const int ox = col >> 1;
    const bool out_lane = !(col & 1) && ox < pg.wo;
    const float *rowp[NR];
    bool row_ok[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int iy = oy0 * 2 - pg.pad_h + r;
        row_ok[r] = iy >= 0 && iy < pg.h;
        rowp[r] = x + (size_t)img * c * in_hw + (size_t)min(max(iy, 0), pg.h - 1) * pg.w;
    }
    const bool padded = pg.pad_h != 0 || pg.pad_w != 0;
    const int groups = (c + 7) >> 3;
    const float inf = __builtin_inff();
    for (int ch = tid; ch < cw * 32; ch += 64 * NW) {
        bn[ch] = bn_scale ? bn_scale[min(ch, c - 1)] : 1.0f;               // (without normalisation y == fma(y, 1, 0))
        bn[cw * 32 + ch] = bn_scale ? bn_shift[min(ch, c - 1)] : 0.0f;
    }
    float asum[R];
#pragma unroll
    for (int r = 0; r < R; ++r) asum[r] = 0.0f;
    for (int g0 = 0; g0 < groups; g0 += NW * side) {
        const int gidx = g0 + slot;
        const int ch0 = min(gidx, groups - 1) * 8, last = c - 1 - ch0, real = gidx < groups ? last + 1 : 0;
        float v[8][NR];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t off = (uint32_t)(ch0 + min(j, last)) * (uint32_t)in_hw + (uint32_t)min(max(xc, 0), pg.w - 1);
#pragma unroll
            for (int r = 0; r < NR; ++r) v[j][r] = rowp[r][off];
        }
        if (g0 == 0) __syncthreads();             // (scale and shift; the loads are on their way)
        uint32_t byte[R];
#pragma unroll
        for (int r = 0; r < R; ++r) byte[r] = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (padded) {
#pragma unroll
                for (int r = 0; r < NR; ++r) v[j][r] = row_ok[r] && in_row ? v[j][r] : -inf;
            }
            const bool ok = j < real;
            const float sc = bn[ch0 + j], sh = bn[cw * 32 + ch0 + j];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float m = __builtin_fmaxf(v[j][2 * r], v[j][2 * r + 1]);
                if (PH == 3) m = __builtin_fmaxf(m, v[j][2 * r + PH - 1]);
                m = __builtin_fmaxf(m, next_lane(m));
                if (PH == 3) m = __builtin_fmaxf(m, next_lane(m));
                m = __builtin_fmaxf(m, -inf);
                if (pg.relu) m = m > 0.0f ? m : 0.0f;
                const float y = __builtin_fmaf(m, sc, sh);
                byte[r] |= (ok && y >= 0.0f ? 1u : 0u) << j;
                asum[r] += ok ? __builtin_fabsf(y) : 0.0f;
            }
        }
        if (gidx < groups && out_lane) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r < rows_out) wbytes[(size_t)(r * pg.wo + ox) * cw * 4 + gidx] = (uint8_t)byte[r];
        }
    }
    if (out_lane) {
#pragma unroll
        for (int r = 0; r < R; ++r) part[slot * npx + r * pg.wo + ox] = asum[r];
    }
    __syncthreads();
    const int live = rows_out * pg.wo, slots = min(groups, NW * side);
    const size_t p0 = ((size_t)img * ho + oy0) * pg.wo;
    for (int p = tid; p < live; p += 64 * NW) {
        float s = part[p];
        for (int q = 1; q < slots; ++q) s += part[q * npx + p];            // fixed order
        A[p0 + p] = s / (float)c;
    }
    const uint32_t *words = reinterpret_cast<const uint32_t *>(wbytes);
    const uint32_t tail_mask = 0xFFFFFFFFu >> (8 * (cw * 4 - groups));      // bytes of the last word no group wrote
    for (int i = tid; i < live * cw; i += 64 * NW) xbits[p0 * cw + i] = words[i] & (i % cw == cw - 1 ? tail_mask : 0xFFFFFFFFu);
}

template <int PH>
static xnor_status launch_pool_rows(const float *x, const float *bn_scale, const float *bn_shift, uint32_t *xbits, float *A, int n, int c,
                                    int ho, const PoolGeom &pg, hipStream_t stream)
{
    const int cw = (c + 31) / 32, groups = (c + 7) / 8, width = pg.w + 2 * pg.pad_w;
    if (width > 64 || (long long)c * pg.h * pg.w >= (1ll << 30)) return XNOR_ERR_UNSUPPORTED;
    int lanes_log2 = 3;
    while ((1 << lanes_log2) < width) ++lanes_log2;
    const int side = 64 >> lanes_log2;
    // One pooled row per workgroup where two leave CUs without one.  Waves: those that the channels fill, up to 8 (several workgroups of 64 to
    // 72 registers then share a CU, one loads while another computes: 64 of 256x27x27 11.7 us, with 16 waves 14.8; 256 of 128x28x28
    // 18.8 / 32.4), 16 where there are CUs to spare (2 of 480x40x40 11.3 / 9.7, 4 of 100x33x33 4.9 / 4.6).
    const int R = (long long)n * ((ho + 1) / 2) < 256 ? 1 : 2, waves = (groups + side - 1) / side;
    const int NW = R == 1 && waves > 8 && (long long)n * ho < 256 ? 16 : waves > 4 ? 8 : 4;
    const int tiles = (ho + R - 1) / R;
    const long long blocks = (long long)n * tiles;
    const size_t lds = (size_t)R * pg.wo * 4 * (cw + NW * side) + (size_t)cw * 64 * 4;
    if (blocks > 0x7ffffff0LL || lds > 48 * 1024) return XNOR_ERR_UNSUPPORTED;
#define XNOR_PR(RR, W) \
    pool_rows_kernel<PH, RR, W><<<dim3((unsigned)blocks), dim3(64 * W), lds, stream>>>(x, bn_scale, bn_shift, xbits, A, c, cw, ho, tiles, (int)blocks, lanes_log2, pg)
    if (R == 1) { if (NW == 16) XNOR_PR(1, 16); else if (NW == 8) XNOR_PR(1, 8); else XNOR_PR(1, 4); }
    else        { if (NW == 8) XNOR_PR(2, 8); else XNOR_PR(2, 4); }
#undef XNOR_PR
    return hip_status(hipGetLastError());
}

xnor_status launch_pool_binactiv(const float *x, const float *bn_scale, const float *bn_shift,
                                 uint32_t *xbits, float *A, int n, int c, int h, int w, int ph, int pw,
                                 int sh, int sw, int pad_h, int pad_w, int relu, hipStream_t stream)
{
    PoolGeom pg;
    pg.h = h; pg.w = w; pg.ph = ph; pg.pw = pw; pg.sh = sh; pg.sw = sw; pg.pad_h = pad_h; pg.pad_w = pad_w;
    pg.relu = relu;
    const int ho = (h + 2 * pad_h - ph) / sh + 1, wo = (w + 2 * pad_w - pw) / sw + 1;
    pg.wo = wo;
    if (ph == pw && (ph == 2 || ph == 3) && sh == 2 && sw == 2 && xbits && A) {
        const xnor_status s = ph == 3 ? launch_pool_rows<3>(x, bn_scale, bn_shift, xbits, A, n, c, ho, pg, stream)
                                      : launch_pool_rows<2>(x, bn_scale, bn_shift, xbits, A, n, c, ho, pg, stream);
        if (s != XNOR_ERR_UNSUPPORTED) return s;
    }
    // LDS staging of the input rows a 64-pixel tile touches (compile-time windows only): at most
    // ceil-ish (64 + wo - 2)/wo + 1 pooled rows, hence (rows - 1)*sh + ph input rows of w floats
    pg.tiles = (ho * wo + 63) / 64;
    pg.px_tile = 64;
    pg.stage = 0;
    if ((ph == 3 && pw == 3) || (ph == 2 && pw == 2)) {
        const long long prows = std::min<long long>(ho, (64 + wo - 2) / wo + 1);
        const long long nfl = std::min<long long>(h, (prows - 1) * sh + ph) * w;
        if (nfl <= 512) pg.stage = (int)nfl;      // 16 waves x 2 channels x 512 floats = 64 KB
    }
    if (ph == 3 && pw == 3) return launch_binactiv_impl<true, 3, 3>(x, bn_scale, bn_shift, xbits, A, n, c, ho * wo, pg, stream);
    if (ph == 2 && pw == 2) return launch_binactiv_impl<true, 2, 2>(x, bn_scale, bn_shift, xbits, A, n, c, ho * wo, pg, stream);
    return launch_binactiv_impl<true>(x, bn_scale, bn_shift, xbits, A, n, c, ho * wo, pg, stream);
}

// K[n][oy][ox] = (1/(kh*kw)) * sum over in-bounds taps of A (sec. 3.2).  One thread per output;
// A is 1/c of the input volume and stays in L2, taps are summed in row-major order.
__global__ __launch_bounds__(256) void boxfilter_kernel(const float *__restrict__ A,
                                                        float *__restrict__ K, ConvGeom g)
{
    const uint32_t m = blockIdx.x * 256u + threadIdx.x;
    if (m >= (uint32_t)g.m_total) return;
    K[m] = box_K(A, g, m);
}

xnor_status launch_boxfilter(const float *A, float *K, const ConvGeom &g, hipStream_t stream)
{
    dim3 grid((unsigned)((g.m_total + 255) / 256)), block(256);
    boxfilter_kernel<<<grid, block, 0, stream>>>(A, K, g);
    return hip_status(hipGetLastError());
}

}  // namespace xnor
