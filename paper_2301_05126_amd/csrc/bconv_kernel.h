// Binary 3x3 convolution (stride 1, pad 1 with -1) for gfx950: im2col-free, on the matrix
// cores.
//
// x[n,y,x,o] = sum_{tap, c} a(n, y+i-1, x+j-1, c) * W[o, tap, c] over +-1 values (paper
// Sec. II-A: convolutional layer of binarized neurons, 2*popcount(xnor) - #bits).  Taps that
// fall outside the image read zero words, i.e. -1 activations, so every output sums exactly
// K = 9*c_in products.
//
// A block of 4 waves (2 x 2) computes (64*TM pixels) x (64*TN output channels) per pixel
// tile and is persistent: it keeps one channel tile and walks over pixel tiles.  The pixels
// of a tile are `ni` images x (th x tw) spatial tile whose input patch, halo included, sits
// in LDS as packed words; the nine taps are read from it with shifted addresses.  Weights
// are resident in LDS when they fit, else they stream through it in chunks of a few taps.
// Every 32-bit word of either operand is expanded in registers into 32 FP4 values +-1.0 and
// multiplied by v_mfma_f32_32x32x64_f8f6f4 (no block scales); all sums are multiples of 1/2
// far below 2^23, so the FP32 accumulators are exact.  Within one MFMA the lower 32 lanes
// supply the first half of a pixel's channel words and the upper 32 lanes the second half
// (same split on the weight side).
//
// The weights are the MFMA's first operand, so a lane owns 16 channels of one pixel, and
// pixels are numbered window-major (four consecutive rows of the implicit GEMM are one 2x2
// window = one lane quad); the step and pool layers fused behind the sums are described in
// conv_epilogue.h.
#ifndef BNN_BCONV_KERNEL_H
#define BNN_BCONV_KERNEL_H
#include "bnn_internal.h"
#include "conv_epilogue.h"
#include "lds_dma.h"

namespace bnn {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

// LDS per block: gfx950 has 160 KB per compute unit and lets one block take all of it; two
// resident blocks per compute unit leave 80 KB each.
constexpr int MAX_SMEM = 80 * 1024;

template <int V> struct WordVec;
template <> struct WordVec<4> { using type = uint4; };
template <> struct WordVec<2> { using type = uint2; };
template <> struct WordVec<1> { using type = uint32_t; };

__device__ __forceinline__ uint32_t vec_word(const uint4 &v, int q) { return q == 0 ? v.x : (q == 1 ? v.y : (q == 2 ? v.z : v.w)); }
__device__ __forceinline__ uint32_t vec_word(const uint2 &v, int q) { return q == 0 ? v.x : v.y; }
__device__ __forceinline__ uint32_t vec_word(const uint32_t &v, int) { return v; }
// operand of a word group's first step (see expand_pair_half for the two-word groups)
template <int V, typename VecT>
__device__ __forceinline__ v8i expand_first(const VecT &v, uint32_t sgn, uint32_t one)
{
    if constexpr (V == 2) {
        const uint2 lo = expand_pair_half(v, 0, 0, sgn, one), hi = expand_pair_half(v, 0, 1, sgn, one);
        v8i r;
        r[0] = (int)lo.x; r[1] = (int)lo.y; r[2] = (int)hi.x; r[3] = (int)hi.y;
        r[4] = 0; r[5] = 0; r[6] = 0; r[7] = 0;
        return r;
    } else {
        return expand_fp4(vec_word(v, 0), sgn, one);
    }
}

__device__ __forceinline__ void vec_set(uint4 &v, int q, uint32_t x) { if (q == 0) v.x = x; else if (q == 1) v.y = x; else if (q == 2) v.z = x; else v.w = x; }
__device__ __forceinline__ void vec_set(uint2 &v, int q, uint32_t x) { if (q == 0) v.x = x; else v.y = x; }
__device__ __forceinline__ void vec_set(uint32_t &v, int, uint32_t x) { v = x; }

// Steps (one MFMA K-slice = one word per lane half) per weight chunk, by words per half.
constexpr int steps_per_chunk(int wph) { return wph == 1 ? 9 : (wph == 2 ? 18 : (wph == 4 ? 12 : (wph == 6 ? 6 : 8))); }

// Whether a block keeps all of its weight chunks in LDS at once: up to 40 KB for any tile
// (C_in <= 256 with 128 output channels), up to 48 KB for the 64-channel tile.
constexpr bool weights_resident(int tm, int tn, int wph)
{
    const int v = wph >= 2 ? 2 : wph;
    const int lsb = 2 * steps_per_chunk(wph) + v;
    const int nchunk = 9 * wph / steps_per_chunk(wph);
    const int bytes = nchunk * 64 * tn * lsb * 4;
    return bytes <= 40 * 1024 || (tm * tn == 1 && bytes <= 48 * 1024);
}

// WDMA: the weight word that a lane delivers with transfer k (0..7) of a chunk.  A chunk buffer's row
// holds 16 words, eight places for each lane half of which the first SPC are used; transfer k of wave
// `wave` fills rows 4 * (wave + 4k) .. +3 of it.  The word's address is voff() + chunk_offset(), the
// latter (and k's rows, where the layer is exact) in the scalar offset.  A scalar offset need not take
// part in the buffer's range check, so a lane that has no word must say so in the vector offset: with
// six words per half, places 6 and 7 would otherwise read the next tap's first words, and behind
// the last tap of the last channel eight bytes past the tensor.
template <int WPH>
struct WeightLane {
    static constexpr int SPC = steps_per_chunk(WPH);
    static constexpr unsigned NONE = 0x80000000u;          // past the end of any weight tensor (< 2 GiB)
    unsigned first;                                        // transfer 0
    bool place, ok[2];                                     // the place is used; the word exists (even / odd chunk)

    __host__ __device__ __forceinline__ WeightLane(int o_blk, int wave, int lane, int cw)
    {
        const int phys = (lane & 15) >> 1, sub = lane & 1;
        const int lw = ((phys ^ ((2 * wave + (lane >> 5)) & 7)) << 1) | sub;    // logical word of the chunk row
        const int hh = lw >> 3, st = lw & 7;
        first = (unsigned)(((o_blk + 4 * wave + (lane >> 4)) * 9 * cw + hh * WPH + st) * 4);
        place = st < SPC;
        ok[0] = place && hh * WPH + st < cw;
        ok[1] = place && hh * WPH + st + (WPH > 8 ? 8 : 0) < cw;
    }
    __host__ __device__ static __forceinline__ unsigned chunk_offset(int chunk, int cw)
    {
        const int s0 = chunk * SPC;
        return (unsigned)(((s0 / WPH) * cw + s0 % WPH) * 4);
    }
    // bytes between the rows of transfers k and k + 1
    __host__ __device__ static __forceinline__ unsigned row_step(int cw) { return (unsigned)(16 * 9 * 4) * (unsigned)cw; }
    // exact: 2 * WPH words per pixel and whole channel tiles, every place's row exists
    __host__ __device__ __forceinline__ unsigned voff_exact() const { return place ? first : NONE; }
    __host__ __device__ __forceinline__ unsigned voff(int chunk, int k, int cw) const
    {
        return (WPH > 8 && (chunk & 1) ? ok[1] : ok[0]) ? first + k * row_step(cw) : NONE;
    }
};

struct TileCoord {
    int group, ty, tx;           // image group, tile row, tile column (LIN: first image, first unit inside it, -)
};

struct ConvGeom {
    int n, h, w, cw;             // input: images, height, width, words per pixel
    int c_out, k_bits;           // outputs, K = 9*c_in
    int lth, ltw;                // log2 of the spatial tile height / width (both >= 1)
    int ni;                      // images per pixel tile; ni * th * tw == pixels per block
    int tiles_x, tiles_y, n_co_tiles;
    int n_ptiles;                // pixel tiles in the layer
    int slots;                   // blocks per channel tile = pixel tiles in flight
    int patch_words;             // LDS words of one patch buffer (rounded up)
    int wexact;                  // WDMA: exactly 2*WPH words per pixel and whole channel tiles
    int dbuf;                    // 1: two patch buffers, the next tile's patch is fetched during the MFMAs
    unsigned mg_pw, mg_ph;       // ceil(2^32 / d) for d = patch width, patch height (staging index math)
    int step_group, step_ty, step_tx;    // `slots` pixel tiles as an (image group, tile row, tile column) increment
    unsigned mg_co, mg_tpg, mg_tx;       // magic_floor of n_co_tiles, tiles per image group, tiles_x
    // linear tiles (LIN)
    int win;                     // 1: a unit is a 2x2 window, 0: a pixel
    int upi, ww;                 // units per image, per row of units
    int step_img, step_u;        // `slots` tiles as an (image, unit) increment
    unsigned mg_upi, mg_ww, mg_hp;       // magic_floor of upi, ww, h + 2
};

// WPH = words per lane half per tap; the layer's cw words per pixel are zero-padded to 2*WPH.
//
// Blocks are persistent: block b owns channel tile b % n_co_tiles for its whole life (so
// thresholds, and the weights when they are resident, are fetched once) and walks the pixel
// tiles slot, slot + slots, ...  The input patch of a tile goes global -> LDS without passing
// through registers (buffer_load ... lds; lanes outside the image or beyond the last image
// address past the buffer's end and deliver zeros, i.e. -1 padding); with two patch buffers
// the next tile's patch is in flight while the current tile is multiplied.
//
// WDMA (wide layers whose weights are not resident): weight chunks also travel global -> LDS
// without passing through registers, into two buffers that alternate; the chunk sequence is cyclic
// over the tiles (weights do not depend on the tile), so the next chunk is always in flight
// behind the current one and a chunk costs one barrier.  Rows are unpadded (16 words, eight for
// each lane half) and their 8-byte units are stored at position unit ^ ((row >> 1) & 7), which keeps
// the 32 rows read by one instruction on distinct banks.  Channels past c_out and words past the
// layer's own address past the end of the weights and arrive as zeros (staging such layers through
// registers, two barriers per chunk, took 39.8 us for 1137 x 7 x 7, 320 -> 184; this takes 25.9).
//
// LIN: a tile is the next 64*TM pixels (2x2 windows when pooling) of the batch in raster order
// instead of a rectangle per image group, so that images of any size fill their tiles: 21 x 21
// images take 441 rows of the implicit GEMM each, 1024 with 16 x 16 rectangles.  The patch is then
// the padded rows (w + 2 pixels; an image has h + 2 of them) that these pixels touch, a pixel's place
// in it is worked out per tile, and the output words are contiguous.  Rectangles stay where the
// image is made of them exactly (no work per tile for the addresses) and where whole rows do not
// fit LDS.  Rectangles / linear tiles, us: 200 x 17 x 17, 224 -> 224 48.0 / 18.5; 105 x 21 x 21, 128 -> 320
// 18.1 / 13.9; 1137 x 7 x 7, 320 -> 184 53.5 / 39.8; 131 x 27 x 31, 256 -> 64 19.2 / 14.7.
template <int TM, int TN, int WPH, bool WDMA, bool LIN>
__global__ __launch_bounds__(256, 2)
void bconv_mfma(const uint32_t *__restrict__ in, const uint32_t *__restrict__ wt, ConvGeom g, EpiArgs ep)
{
    constexpr int BN = 64 * TN;
    constexpr int BW = 2 * TN;                         // packed output words per pixel of a block
    constexpr int CWP = 2 * WPH;                       // padded words per pixel
    constexpr int V = WPH >= 2 ? 2 : WPH;              // words per LDS access
    constexpr int SPC = steps_per_chunk(WPH);
    constexpr int NCHUNK = 9 * WPH / SPC;
    constexpr int LSB = WDMA ? 16 : 2 * SPC + V;       // weight row stride (words); padded: LSB/V is odd
    constexpr int UPRW = 2 * SPC / V;                  // weight units per row per chunk
    constexpr int STG = (BN * UPRW + 255) / 256;       // weight units per thread per chunk
    constexpr int NVG = SPC / V;                       // V-step groups per chunk
    constexpr bool RES = !WDMA && weights_resident(TM, TN, WPH);
    constexpr int NBUF = RES ? NCHUNK : (WDMA ? 2 : 1);
    static_assert(!WDMA || (SPC <= 8 && V == 2 && BN == 128), "weight DMA layout: 16-word rows, 128 rows");
    // word groups in registers: the current one, the next, and with an odd number of groups per chunk
    // a third place, so that every chunk starts with the same one
    constexpr int NSLOT = NVG % 2 != 0 && NCHUNK > 1 ? 3 : 2;
    static_assert(NSLOT == 2 || NVG == 3, "a chunk's groups and the next chunk's first one have places of their own");
    static_assert(SPC % 2 == 0 || NCHUNK == 1, "operand pipeline across chunks: buffer parity");
    using vec_t = typename WordVec<V>::type;

    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *Bs = reinterpret_cast<uint32_t *>(smem);                 // [NBUF][BN][LSB] weights
    float *Ts = reinterpret_cast<float *>(Bs + NBUF * BN * LSB);       // [BN] accumulator start values
    uint32_t *Os = reinterpret_cast<uint32_t *>(Ts + BN);              // [2][64*TM][BW] output tiles
    uint32_t *Ps = Os + 2 * 64 * TM * BW;                              // [1 or 2][patch_words]

    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;

    // XCD-aware order: hardware deals consecutive block ids round-robin to the 8 XCDs (one L2
    // each); renumber so that blocks working on the same pixel tile (its channel tiles) share
    // an XCD and the patch is fetched from HBM once.
    int bid = blockIdx.x;
    if ((gridDim.x & 7) == 0) bid = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int slot = div_by(bid, g.n_co_tiles, g.mg_co);
    const int co_tile = bid - slot * g.n_co_tiles;
    const int th = 1 << g.lth, tw = 1 << g.ltw;
    const int o_blk = co_tile * BN;
    const int pw = LIN ? g.w + 2 : tw + 2, ph = LIN ? g.h + 2 : th + 2;
    const int tiles_per_group = g.tiles_x * g.tiles_y;
    const int UB = LIN ? (g.win ? 16 * TM : 64 * TM) : 0;            // units per tile
    // image row of a unit (first row of a window), relative to its image
    auto unit_row = [&](int rem) { return div_by(rem, g.ww, g.mg_ww) << g.win; };

    // ---- per-channel step parameters and (if resident) all weight chunks: once per block,
    // requested further down, behind the first patch, so that all of it is in flight together
    const int corr = 9 * CWP * 32 - g.k_bits;          // padded positions all counted as +1
    StepWords<TN> sw;
    const float *Tw = Ts + wn * TN * 32;               // this wave's channels

    // weight staging: LDS row = [half 0: SPC words][half 1: SPC words]; the word of
    // (half, step) is W[o][tap][half*WPH + cwi] with tap = step / WPH, cwi = step % WPH.
    vec_t pb[STG];
    const bool wvec_ok = (g.cw % V) == 0;
    // A thread's units keep their row and position inside the chunk; per chunk only a uniform
    // (tap, word) offset is added.  (step = chunk * SPC + vg * V splits into a chunk part and a
    // unit part without carry because SPC is a multiple of WPH or the other way round.)
    static_assert(SPC % WPH == 0 || WPH % SPC == 0, "chunk and unit parts of a step index add without carry");
    int wu_off[STG], wu_cw[STG];                       // word offset / word inside the pixel, chunk 0
    bool wu_row[STG];
    if (!WDMA) {
#pragma unroll
        for (int r = 0; r < STG; ++r) {
            const int idx = t + 256 * r;
            const int row = idx / UPRW, u = idx % UPRW;
            const int hh = u / NVG, s0 = (u % NVG) * V;
            const int tapr = WPH <= SPC ? s0 / WPH : 0, cwir = WPH <= SPC ? s0 % WPH : s0;
            const int o = o_blk + row;
            wu_row[r] = row < BN && o < g.c_out;
            wu_cw[r] = hh * WPH + cwir;
            wu_off[r] = (o * 9 + tapr) * g.cw + wu_cw[r];
        }
    }
    auto load_w_to = [&](int chunk, vec_t (&dst)[STG]) {
        // Branch-free inside each loop, so that all loads of a chunk are in flight together:
        // rows or words that do not exist read the first weight word and are zeroed afterwards.
        const int sc = chunk * SPC;
        const int cwic = sc % WPH;
        const int coff = (sc / WPH) * g.cw + cwic;
        auto unit = [&](int r, bool &row_ok, int &cwpos) {
            cwpos = wu_cw[r] + cwic;
            row_ok = wu_row[r];
            return wu_off[r] + coff;
        };
        if (wvec_ok) {
#pragma unroll
            for (int r = 0; r < STG; ++r) {
                bool row_ok;
                int cwpos;
                const int off = unit(r, row_ok, cwpos);
                const bool ok = row_ok && cwpos < g.cw;
                vec_t v = *reinterpret_cast<const vec_t *>(wt + (unsigned)(ok ? off : 0));
#pragma unroll
                for (int q = 0; q < V; ++q) vec_set(v, q, ok ? vec_word(v, q) : 0u);
                dst[r] = v;
            }
        } else {
#pragma unroll
            for (int r = 0; r < STG; ++r) {
                bool row_ok;
                int cwpos;
                const int off = unit(r, row_ok, cwpos);
                vec_t v;
#pragma unroll
                for (int q = 0; q < V; ++q) {
                    const bool ok = row_ok && cwpos + q < g.cw;
                    const uint32_t x = wt[(unsigned)(ok ? off + q : 0)];
                    vec_set(v, q, ok ? x : 0u);
                }
                dst[r] = v;
            }
        }
    };
    auto store_w_from = [&](int buf, const vec_t (&src)[STG]) {
#pragma unroll
        for (int r = 0; r < STG; ++r) {
            const int idx = t + 256 * r;
            const int row = idx / UPRW, u = idx % UPRW;
            if (row < BN) *reinterpret_cast<vec_t *>(Bs + (buf * BN + row) * LSB + u * V) = src[r];
        }
    };
    auto load_w = [&](int chunk) { load_w_to(chunk, pb); };
    auto store_w = [&](int buf) { store_w_from(buf, pb); };

    // WDMA: a chunk's transfers (which word a lane delivers: see WeightLane)
    v4i wd_rsrc = make_raw_rsrc(wt, (unsigned)g.c_out * 9u * (unsigned)g.cw * 4u);
    const WeightLane<WPH> wd(o_blk, wave, lane, g.cw);
    const unsigned wd_exact = wd.voff_exact();
    auto dma_w = [&](int chunk, int buf) {
        // (wave-uniform; read through readfirstlane so that it reaches the transfer's scalar
        // operand in a scalar register whatever the compiler makes of the chunk index)
        const unsigned soff0 = (unsigned)__builtin_amdgcn_readfirstlane((int)wd.chunk_offset(chunk, g.cw));
        const unsigned dst = (unsigned)(size_t)(__attribute__((address_space(3))) uint32_t *)(Bs + buf * BN * LSB) +
                             (unsigned)__builtin_amdgcn_readfirstlane(wave) * 256u;
        const unsigned rows16 = wd.row_step(g.cw);
        if (g.wexact) {
#pragma unroll
            for (int k = 0; k < 8; ++k) lds_dma4_soff(wd_rsrc, dst + k * 1024u, wd_exact, soff0 + k * rows16);
        } else {
            // the row in the vector offset, where the range check sees it
#pragma unroll
            for (int k = 0; k < 8; ++k)
                lds_dma4_soff(wd_rsrc, dst + k * 1024u, wd.voff(chunk, k, g.cw), soff0);
        }
    };
    // this lane's read offsets (words) inside a weight row, per V-step group
    int wd_boff[NVG];
#pragma unroll
    for (int vg = 0; vg < NVG; ++vg) wd_boff[vg] = (((half * 4 + vg) ^ ((l32 >> 1) & 7)) << 1);

    // ---- patch fetch, global -> LDS directly.  Unit = 16 bytes (a whole-pixel multiple) when
    // a pixel is a whole number of them, else one word.
    const bool wide = CWP % 4 == 0 && (g.cw & 3) == 0;
    auto fetch_patch = [&](const TileCoord &tc, int buf) {
        const int img0 = LIN ? tc.group : tc.group * g.ni;
        const int y0 = LIN ? unit_row(tc.ty) : tc.ty * th, x0 = LIN ? 0 : tc.tx * tw;
        int imgs = g.n - img0, rows = 0;
        if (LIN) {                      // padded rows from above the first pixel's to below the last one's
            const int il = div_by(tc.ty + UB - 1, g.upi, g.mg_upi);
            rows = il * ph + unit_row(tc.ty + UB - 1 - il * g.upi) + g.win + 3 - y0;
            imgs = min(il + 1, imgs);
        } else {
            imgs = min(g.ni, imgs);
        }
        const uint32_t *base = in + (int64_t)img0 * g.h * g.w * g.cw;
        const unsigned bytes = (unsigned)imgs * g.h * g.w * g.cw * 4;
        const v4i rsrc = make_raw_rsrc(base, bytes);
        // LDS byte address of the destination buffer
        const unsigned dst = (unsigned)(size_t)(__attribute__((address_space(3))) uint32_t *)(Ps + buf * g.patch_words);
        const int upp = wide ? CWP / 4 : CWP;               // units per pixel
        const int total = (LIN ? rows : g.ni * ph) * pw * upp;
        for (int b0 = 0; b0 < total; b0 += 256) {
            const int idx = b0 + t;
            // idx -> (image, row, column, unit) of the patch; divisions by multiply-high
            const int p0 = idx / upp, u = idx - p0 * upp;
            const int p1 = (int)__umulhi((unsigned)p0, g.mg_pw), px = p0 - p1 * pw;
            const int il = LIN ? div_by(y0 + p1, ph, g.mg_hp) : (int)__umulhi((unsigned)p1, g.mg_ph);
            const int py = p1 - il * ph;
            const int y = y0 + py - 1, x = x0 + px - 1;
            const bool inside = y >= 0 && y < g.h && x >= 0 && x < g.w && (wide ? u * 4 : u) < g.cw;
            unsigned voff = 0x80000000u;                    // past the end of the buffer: zeros
            if (inside) voff = (unsigned)(((il * g.h + y) * g.w + x) * g.cw) * 4u + (unsigned)u * (wide ? 16u : 4u);
            const unsigned wave_base = (unsigned)__builtin_amdgcn_readfirstlane(b0 + wave * 64);
            if (idx < total) {
                if (wide) lds_dma16(rsrc, dst + wave_base * 16u, voff);
                else lds_dma4(rsrc, dst + wave_base * 4u, voff);
            }
        }
    };

    // ---- this lane's pixels: implicit-GEMM row p = 4 * window + (2*dy + dx)
    int pixoff[TM];
    // LIN: of the tile that starts at unit u0 of its first image
    auto place_pixels = [&](int u0) {
        const int y0 = unit_row(u0);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int p = wm * TM * 32 + i * 32 + l32;
            const int u = u0 + (g.win ? p >> 2 : p);
            const int il = div_by(u, g.upi, g.mg_upi), rem = u - il * g.upi;
            const int ry = div_by(rem, g.ww, g.mg_ww), rx = rem - ry * g.ww;
            const int y = g.win ? 2 * ry + ((p >> 1) & 1) : ry, x = g.win ? 2 * rx + (p & 1) : rx;
            pixoff[i] = ((il * ph + y - y0) * pw + x) * CWP + half * WPH;
        }
    };
    if (!LIN) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int p = wm * TM * 32 + i * 32 + l32;
            const int wq = p >> 2, sub = p & 3;
            const int wx = wq & ((tw >> 1) - 1);
            const int wy = (wq >> (g.ltw - 1)) & ((th >> 1) - 1);
            const int il = wq >> (g.ltw - 1 + g.lth - 1);
            const int py = 2 * wy + (sub >> 1), px = 2 * wx + (sub & 1);
            pixoff[i] = ((il * ph + py) * pw + px) * CWP + half * WPH;
        }
    }
    const int browoff = (wn * TN * 32 + l32) * LSB + half * SPC;

    uint32_t sgn = 0x88888888u, one = 0x22222222u;
    asm volatile("" : "+s"(sgn));
    asm volatile("" : "+v"(one));
    constexpr int DPM = (4 * (TM + TN) + TM * TN - 1) / (TM * TN);   // operand dwords made per MFMA

    // tile coordinates of the previous, current and next pixel tile of this block; a step of
    // `slots` tiles is a fixed (group, y, x) increment with carries
    TileCoord step, prev, cur, next;
    step.group = g.step_group; step.ty = g.step_ty; step.tx = g.step_tx;
    if (LIN) {
        next.group = div_by(slot * UB, g.upi, g.mg_upi);
        next.ty = slot * UB - next.group * g.upi;
        next.tx = 0;
    } else {
        next.group = div_by(slot, tiles_per_group, g.mg_tpg);
        next.ty = div_by(slot - next.group * tiles_per_group, g.tiles_x, g.mg_tx);
        next.tx = slot - next.group * tiles_per_group - next.ty * g.tiles_x;
    }
    prev = cur = next;
    auto advance = [&](TileCoord &c) {
        if (LIN) {
            c.ty += g.step_u;
            c.group += g.step_img;
            if (c.ty >= g.upi) { c.ty -= g.upi; ++c.group; }
            return;
        }
        c.tx += step.tx;
        if (c.tx >= g.tiles_x) { c.tx -= g.tiles_x; ++c.ty; }
        c.ty += step.ty;
        if (c.ty >= g.tiles_y) { c.ty -= g.tiles_y; ++c.group; }
        c.group += step.group;
    };
    auto tile_pos = [&](const TileCoord &c) {
        TilePos pos;
        pos.n = g.n; pos.h = g.h; pos.w = g.w; pos.c_out = g.c_out;
        pos.lth = g.lth; pos.ltw = g.ltw; pos.img0 = c.group * g.ni; pos.y0 = c.ty * th; pos.x0 = c.tx * tw;
        return pos;
    };

    CopyLane copy_lane;
    if (!LIN) copy_lane = make_copy_lane(64 * TM, tile_pos(next), ep.pool, t);
    // packed words of a finished tile, LDS -> global
    auto copy_out = [&](const uint32_t *tile, const TileCoord &c) {
        if (!LIN) {
            conv_tile_copy_out<BW>(tile, copy_lane, o_blk >> 5, tile_pos(c), ep);
        } else {
            const int cwo = (g.c_out + 31) >> 5;
            const int64_t left = (int64_t)(g.n - c.group) * g.upi - c.ty;      // units from the tile's first
            if (t < UB && t < left)
                copy_words<BW>(tile + t * BW, ep.packed + ((int64_t)c.group * g.upi + c.ty + t) * cwo + (o_blk >> 5),
                               cwo, o_blk >> 5);
        }
    };
    if (slot < g.n_ptiles) fetch_patch(next, 0);
    if (WDMA && slot < g.n_ptiles) dma_w(0, 0);
    // resident weights (at most 48 registers per thread), flips and thresholds: every load is
    // issued before the first one is waited for, one memory latency for all of them
    if (RES) {
        vec_t pall[NCHUNK][STG];
#pragma unroll
        for (int c = 0; c < NCHUNK; ++c) load_w_to(c, pall[c]);
        if (ep.packed) sw = load_step_words<TN>(ep, o_blk + wn * TN * 32, l32, g.c_out);
        stage_bias_f32(ep, o_blk, BN, g.c_out, g.k_bits + 1, corr, Ts, t);
#pragma unroll
        for (int c = 0; c < NCHUNK; ++c) store_w_from(c, pall[c]);
    } else {
        if (ep.packed) sw = load_step_words<TN>(ep, o_blk + wn * TN * 32, l32, g.c_out);
        stage_bias_f32(ep, o_blk, BN, g.c_out, g.k_bits + 1, corr, Ts, t);
    }
    int cc = 0;                                            // chunks done so far (WDMA buffer parity)

    // The packed words of a tile go to one of two LDS output tiles and are copied to global
    // memory after the next tile's barrier, so the stores drain while the next tile is
    // multiplied and the block needs one barrier per tile.
    // The tile loop starts 4 bytes behind a 32-byte boundary, whatever the code before it: where the layer's
    // multiplies fit one or two rounds its speed depends on that (256 x 128 tile, four words per pixel,
    // us at the eight places of a word in 32 bytes: 350 x 16 x 16, 128 -> 256 15.06 here, 15.13 .. 15.50
    // elsewhere; at 1024 x 16 x 16, 128 -> 128 15.22 and 15.27 .. 15.65).
    asm volatile(".p2align 5\n\t.fill 1, 4, 0xbf800000");        // s_nop 0
    int it = 0;
    for (int ptile = slot; ptile < g.n_ptiles; ptile += g.slots, ++it) {
        const int buf = g.dbuf ? (it & 1) : 0;
        const uint32_t *Pc = Ps + buf * g.patch_words;
        uint32_t *Oc = Os + (it & 1) * (64 * TM * BW);
        prev = cur;
        cur = next;
        advance(next);
        if (!RES && !WDMA) load_w(0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this tile's patch (and first weight chunk) has landed
        __syncthreads();                                      // ... for every wave; previous tile fully consumed
        if (g.dbuf && ptile + g.slots < g.n_ptiles) fetch_patch(next, buf ^ 1);
        if (ep.packed && it > 0)
            copy_out(Os + ((it - 1) & 1) * (64 * TM * BW), prev);
        if (LIN) place_pixels(cur.ty);

        __builtin_amdgcn_s_setprio(1);                        // the multiply phase outranks another wave's epilogue
        // accumulators start at the channels' biases (see stage_bias_f32)
        v16f acc[TM][TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const v16f b16 = load_bias16<v16f>(Tw + j * 32, half);
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[i][j] = b16;
        }

        // Raw words of a V-step group (TM pixels' words, TN channels' words) and the expanded
        // operands of the current and the next MFMA step.  The pipeline "read words, expand
        // them, multiply" runs across chunk borders where the data allows it (XA: pixel words
        // always, the patch is resident; XB: channel words only when the weights are resident).
        constexpr bool XA = RES || WDMA, XB = RES;
        vec_t ra[NSLOT][TM], rb[NSLOT][TN];
        v8i a[2][TM], b[2][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 4; q < 8; ++q) a[0][i][q] = a[1][i][q] = 0;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 4; q < 8; ++q) b[0][j][q] = b[1][j][q] = 0;
        auto load_a = [&](int c, int vg, int slot2) {
            const int s = c * SPC + vg * V;
            const int tap = s / WPH, cwi = s % WPH;
            const int ti = tap / 3, tj = tap - ti * 3;
            const int aoff = (ti * pw + tj) * CWP + cwi;
#pragma unroll
            for (int i = 0; i < TM; ++i) ra[slot2][i] = *reinterpret_cast<const vec_t *>(Pc + pixoff[i] + aoff);
        };
        auto load_b = [&](const uint32_t *Bc, int vg, int slot2) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
                rb[slot2][j] = *reinterpret_cast<const vec_t *>(
                    WDMA ? Bc + (wn * TN * 32 + j * 32 + l32) * LSB + wd_boff[vg] : Bc + browoff + j * 32 * LSB + vg * V);
        };
        if (XA) {                                           // pixel operands of the tile's first step
            load_a(0, 0, 0);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const v8i e = expand_first<V>(ra[0][i], sgn, one);
#pragma unroll
                for (int q = 0; q < 4; ++q) a[0][i][q] = e[q];
            }
        }

        // resident weights: the chunk loop is unrolled too (straight-line code keeps the operand
        // pipeline in registers without copies)
        constexpr int CUNROLL = RES ? NCHUNK : 1;
#pragma unroll CUNROLL
        for (int c = 0; c < NCHUNK; ++c) {
            if (WDMA) {
                if (c > 0) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this chunk has landed
                    __syncthreads();              // ... for every wave; previous chunk consumed
                }
                // next chunk of the cyclic sequence into the other buffer
                if (c + 1 < NCHUNK || ptile + g.slots < g.n_ptiles) dma_w(c + 1 < NCHUNK ? c + 1 : 0, (cc + 1) & 1);
            } else if (!RES) {
                if (c > 0) __syncthreads();       // previous chunk consumed
                store_w(0);
                __syncthreads();
                if (c + 1 < NCHUNK) load_w(c + 1);
            }
            const uint32_t *Bc = RES ? Bs + c * BN * LSB : (WDMA ? Bs + (cc & 1) * BN * LSB : Bs);
            const uint32_t *Bn = Bc + BN * LSB;            // next chunk's weights (resident weights only)
            if (WDMA) ++cc;
            const bool more = c + 1 < NCHUNK;

            // operands of the chunk's first step that did not come from the previous chunk
            if (!XA) {
                load_a(c, 0, 0);
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const v8i e = expand_first<V>(ra[0][i], sgn, one);
#pragma unroll
                    for (int q = 0; q < 4; ++q) a[0][i][q] = e[q];
                }
            }
            if (!XB || c == 0) {
                load_b(Bc, 0, 0);
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const v8i e = expand_first<V>(rb[0][j], sgn, one);
#pragma unroll
                    for (int q = 0; q < 4; ++q) b[0][j][q] = e[q];
                }
            }
            // The instruction order below is the issue order (scheduling barriers pin it): the
            // LDS reads of the next word group, then each MFMA followed by its share of the
            // next step's operand dwords, so that VALU work runs in the shadow of the MFMAs.
#pragma unroll
            for (int st = 0; st < SPC; ++st) {
                const int cur_s = st & 1, nxt = cur_s ^ 1;
                const int vg = st / V, q = st % V;
                const bool last_group = vg + 1 == NVG;
                if (q == 0) {
                    if (!last_group) {
                        load_a(c, vg + 1, (vg + 1) % NSLOT);
                        load_b(Bc, vg + 1, (vg + 1) % NSLOT);
                    } else if (more) {                    // first group of the next chunk
                        if (XA) load_a(c + 1, 0, 0);
                        if (XB) load_b(Bn, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                const bool in_chunk = st + 1 < SPC;
                const int vg1 = in_chunk ? (st + 1) / V : 0, q1 = in_chunk ? (st + 1) % V : 0;
                const int sl1 = vg1 % NSLOT;
                // (streamed weights: the chunk index is a run-time value, and the last chunk expands
                // stale words into operands that the next tile overwrites, rather than branching)
                const bool next_a = in_chunk || (XA && (WDMA || more)), next_b = in_chunk || (XB && more);
                uint2 pend[2 * (TM + TN)];                // shifted pairs awaiting their masks
#pragma unroll
                for (int k = 0; k < TM * TN; ++k) {
                    const int i = k / TN, j = k % TN;
                    // weights first: accumulator rows = channels, columns (lanes) = pixels
                    // (zero scale operands select the instruction form without block scales)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        b[cur_s][j], a[cur_s][i], acc[i][j], 4, 4, 0, 0, 0, 0);
                    if constexpr (V == 2) {
                        // Word pairs: TM + TN pairs, two (shift, mask, mask) items each.  An item's
                        // masks come one MFMA after its shift (no VALU instruction waits for the one
                        // before it); with a single MFMA per step both fall behind that one.
                        constexpr int NIT = 2 * (TM + TN), NM = TM * TN, LAG = NM > 1 ? 1 : 0;
#pragma unroll
                        for (int t2 = 0; t2 < NIT; ++t2) {
                            const int ks = t2 * (NM - LAG) / NIT;            // MFMA the shift follows
                            const int wi = t2 >> 1, dp = t2 & 1;
                            if (!(wi < TM ? next_a : next_b)) continue;
                            if (ks == k) pend[t2] = shift_pair_half(wi < TM ? ra[sl1][wi] : rb[sl1][wi - TM], q1, dp);
                            if (ks + LAG == k) {
                                const uint2 e = mask_pair(pend[t2], sgn, one);
                                if (wi < TM) {
                                    a[nxt][wi][2 * dp] = (int)e.x;
                                    a[nxt][wi][2 * dp + 1] = (int)e.y;
                                } else {
                                    b[nxt][wi - TM][2 * dp] = (int)e.x;
                                    b[nxt][wi - TM][2 * dp + 1] = (int)e.y;
                                }
                            }
                        }
                    } else {
#pragma unroll
                        for (int d = k * DPM; d < (k + 1) * DPM && d < 4 * (TM + TN); ++d) {
                            const int wi = d >> 2, part = d & 3;
                            if (wi < TM) {
                                if (next_a) a[nxt][wi][part] = (int)expand_part(vec_word(ra[sl1][wi], q1), part, sgn, one);
                            } else {
                                if (next_b)
                                    b[nxt][wi - TM][part] = (int)expand_part(vec_word(rb[sl1][wi - TM], q1), part, sgn, one);
                            }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }

        // ---- epilogue (shared with the first layer)
        __builtin_amdgcn_s_setprio(0);
        if (ep.preact) {
            auto getx = [&](int i, int j, int r) {
                return (int)(acc[i][j][r] - Tw[j * 32 + (r >> 2) * 8 + half * 4 + (r & 3)]) - corr;
            };
            if (!LIN) {
                conv_tile_store_preact<TM, TN>(getx, wm * TM * 32, o_blk + wn * TN * 32, l32, half, tile_pos(cur),
                                               ep.preact);
            } else {
                int row = wm * TM * 32 + l32;
                asm volatile("" : "+v"(row));             // (see conv_tile_store_preact)
                auto getpix = [&](int i) -> int64_t {
                    const int p = row + i * 32;
                    const int u = cur.ty + (g.win ? p >> 2 : p);
                    if (u >= (int64_t)(g.n - cur.group) * g.upi) return -1;
                    if (!g.win) return (int64_t)cur.group * g.upi + u;
                    const int il = div_by(u, g.upi, g.mg_upi), rem = u - il * g.upi;
                    const int ry = div_by(rem, g.ww, g.mg_ww), rx = rem - ry * g.ww;
                    return ((int64_t)(cur.group + il) * g.h + 2 * ry + ((p >> 1) & 1)) * g.w + 2 * rx + (p & 1);
                };
                conv_store_preact<TM, TN>(getx, getpix, o_blk + wn * TN * 32, half, g.c_out, ep.preact);
            }
        }
        if (ep.packed) {
            // bits -> LDS tile [output pixel][2*TN words]; one vector store per pixel later
            auto gets = [&](int i, int j, int r) { return acc[i][j][r]; };
            conv_tile_step_to_lds<TM, TN>(gets, wm * TM * 32, wn * TN, BW, l32, half, sw,
                                          ep.pool, ep.pool_first != 0, Oc);
        }
        if (!g.dbuf && ptile + g.slots < g.n_ptiles) {
            __syncthreads();                                  // every wave is done with the only patch buffer
            fetch_patch(next, 0);
        }
    }
    if (ep.packed && it > 0) {
        __syncthreads();
        copy_out(Os + ((it - 1) & 1) * (64 * TM * BW), cur);
    }
}

template <int TM, int TN, int WPH, bool WDMA>
bool make_geom(int n, int h, int w, int c_in, int c_out, bool win, bool lin, ConvGeom &g, size_t &smem)
{
    constexpr int V = WPH >= 2 ? 2 : WPH;
    constexpr int LSB = WDMA ? 16 : 2 * steps_per_chunk(WPH) + V;
    constexpr int NBUF = WDMA ? 2 : (weights_resident(TM, TN, WPH) ? 9 * WPH / steps_per_chunk(WPH) : 1);
    // weights by DMA: byte offsets (of the last channel tile's missing rows too) below 2^31
    if (WDMA && ((int64_t)c_out + 64 * TN) * 9 * ((c_in + 31) / 32) * 4 >= 0x7fffffffLL) return false;
    g.wexact = (c_in + 31) / 32 == 2 * WPH && c_out % (64 * TN) == 0;
    g.n = n; g.h = h; g.w = w;
    g.cw = (c_in + 31) / 32;
    g.c_out = c_out;
    g.k_bits = 9 * c_in;
    const TileShape ts = make_tile_shape(h, w, 64 * TM);
    g.ltw = ts.ltw; g.lth = ts.lth; g.ni = ts.ni;
    g.tiles_x = ts.tiles_x; g.tiles_y = ts.tiles_y;
    g.n_co_tiles = (c_out + 64 * TN - 1) / (64 * TN);
    const int sh = win ? 1 : 0;
    const int ub = 64 * TM >> (2 * sh);                      // LIN: units per tile
    int64_t ptiles;
    int imgs, pwords;                                        // images a patch can touch, its words
    if (lin) {
        if (h > 1024 || w > 1024) return false;
        g.win = sh; g.upi = (h >> sh) * (w >> sh); g.ww = w >> sh;
        ptiles = ((int64_t)n * g.upi + ub - 1) / ub;
        // rows of units a tile can touch, rows of pixels, plus two padded rows around them and two more
        // at every image border inside the tile
        const int urows = (ub - 1 + g.ww - 1) / g.ww + 1, cross = (ub - 1 + g.upi - 1) / g.upi;
        imgs = cross + 1;
        const int64_t pixels = (int64_t)((urows << sh) + 2 + 2 * cross) * (w + 2);
        if (pixels > 16384) return false;
        pwords = (int)pixels * (2 * WPH);
    } else {
        g.win = 0; g.upi = g.ww = 1;
        ptiles = (int64_t)ts.tiles_x * ts.tiles_y * ((n + ts.ni - 1) / ts.ni);
        imgs = ts.ni;
        pwords = ts.ni * ((1 << ts.lth) + 2) * ((1 << ts.ltw) + 2) * (2 * WPH);
    }
    if (ptiles > 0x3fffffffLL || (int64_t)imgs * h * w * g.cw * 4 >= 0x7fffffffLL) return false;
    if (((int64_t)c_out + 64 * TN) * 9 * g.cw >= 0x7fffffffLL) return false;     // 32-bit weight word offsets
    g.n_ptiles = (int)ptiles;
    // exact for dividends below 2^16 (a patch has at most a few thousand units)
    const int pw = lin ? w + 2 : (1 << ts.ltw) + 2, ph = lin ? h + 2 : (1 << ts.lth) + 2;
    g.mg_pw = (unsigned)((0x100000000ULL + pw - 1) / pw);
    g.mg_ph = (unsigned)((0x100000000ULL + ph - 1) / ph);
    g.mg_hp = magic_floor(ph);
    // one patch buffer: pixels x padded words, rounded up to a wave's worth of 16-byte units
    g.patch_words = (pwords + 255) & ~255;
    const size_t fixed = (size_t)NBUF * 64 * TN * LSB * 4 + 64 * TN * 4 + (size_t)2 * 64 * TM * 2 * TN * 4;
    g.dbuf = (fixed + 2 * (size_t)g.patch_words * 4 <= (size_t)MAX_SMEM) ? 1 : 0;
    smem = fixed + (size_t)(g.dbuf ? 2 : 1) * g.patch_words * 4;
    // persistent grid: two resident blocks per compute unit, a whole number of channel-tile sets
    int slots = 512 / g.n_co_tiles;
    if (slots < 1) slots = 1;
    if (slots > g.n_ptiles) slots = g.n_ptiles;
    g.slots = slots;
    const int tpg = ts.tiles_x * ts.tiles_y;
    g.step_group = slots / tpg;
    g.step_ty = (slots - g.step_group * tpg) / ts.tiles_x;
    g.step_tx = slots - g.step_group * tpg - g.step_ty * ts.tiles_x;
    g.step_img = slots * ub / g.upi;
    g.step_u = slots * ub - g.step_img * g.upi;
    g.mg_co = magic_floor(g.n_co_tiles);
    g.mg_tpg = magic_floor(tpg);
    g.mg_tx = magic_floor(ts.tiles_x);
    g.mg_upi = magic_floor(g.upi);
    g.mg_ww = magic_floor(g.ww);
    return smem <= (size_t)MAX_SMEM;
}

// Estimated ticks of a layer's multiply phase on one tiling: the tiles that the busiest compute unit
// takes, times a tile's MFMAs per wave, times the ticks of an MFMA with the operand expansion of this
// tile shape beside it (5.5 vector instructions per word and TM + TN words per TM * TN MFMAs).  Two
// resident blocks hide each other's expansion up to 4 ticks per instruction (4 x 2: 33 ticks per MFMA
// as measured; 1 x 1: 56), a block alone pays more (2 x 2: 41, 1 x 1: 69).  A tile's epilogue and its
// barriers come on top, twice for a block alone; a last tile whose neighbour block has none is alone too
// (counted as half of a pair, it sent 23 x 19 x 24, 64 -> 256 to the tiling that takes 6.2 us, not 5.5).
// Before the first tile a block fetches its channels' weights, 100 ticks for 64 channels and two words.
template <int TM, int TN, int WPH>
double conv_cost(const ConvGeom &g, bool lin)
{
    constexpr double ops = 5.5 * (TM + TN) / (TM * TN);
    constexpr double pair = 12 + 4 * ops > 33 ? 12 + 4 * ops : 33;
    constexpr double lone = 12 + 5.2 * ops > 33 ? 12 + 5.2 * ops : 33;
    constexpr double mfma = TM * TN * 9 * WPH;
    constexpr double over = 300 + 150.0 * TM * TN;
    constexpr double paired = mfma * pair + over, alone = mfma * lone + 2 * over;       // a tile's ticks
    constexpr double prologue = 100.0 * TN * WPH;
    const int blocks = g.slots * g.n_co_tiles;
    const double addr = lin ? 1.08 : 1.0;
    if (blocks <= 256) return prologue + addr * ((g.n_ptiles + g.slots - 1) / g.slots) * alone;
    // blocks b and b + 256 share a compute unit; the first `rest` blocks have one tile more
    const int full = g.n_ptiles / g.slots, rest = (g.n_ptiles - full * g.slots) * g.n_co_tiles;
    return prologue + addr * (2 * full * paired + (rest > 256 ? 2 * paired : (rest > 0 ? alone : 0)));
}

// Rectangular or linear tiles, whichever cost less; working out a linear tile's addresses is some 8 %
// of a tile (measured where both tilings take the same number of rounds: 28 x 28 images 64 -> 64 at
// batch 256 11.4 us with rectangles and 12.0 with linear tiles, 449 x 12 x 31 17.0 and 17.8).
// Returns the estimated cost, or a negative number if neither fits; *lin says which.
template <int TM, int TN, int WPH, bool WDMA>
double pick_geom(int n, int h, int w, int c_in, int c_out, bool win, ConvGeom &g, size_t &smem, bool *lin)
{
    ConvGeom gl;
    size_t sl;
    const bool rect_ok = make_geom<TM, TN, WPH, WDMA>(n, h, w, c_in, c_out, win, false, g, smem);
    const bool lin_ok = make_geom<TM, TN, WPH, WDMA>(n, h, w, c_in, c_out, win, true, gl, sl);
    const double rect = rect_ok ? conv_cost<TM, TN, WPH>(g, false) : -1;
    const double line = lin_ok ? conv_cost<TM, TN, WPH>(gl, true) : -1;
    *lin = lin_ok && (!rect_ok || line < rect);
    if (*lin) { g = gl; smem = sl; }
    return *lin ? line : rect;
}

template <int TM, int TN, int WPH, bool WDMA, bool LIN>
bnn_status launch_geom(const uint32_t *in, const uint32_t *wt, const ConvGeom &g, size_t smem, const EpiArgs &ep,
                       hipStream_t s)
{
    const unsigned blocks = (unsigned)(g.slots * g.n_co_tiles);
    if (smem > 64 * 1024) {          // above the default limit of dynamic LDS: opt in, once per kernel and device
        static PerDevice raised;
        const hipError_t e = raised.run([] {
            return hipFuncSetAttribute((const void *)bconv_mfma<TM, TN, WPH, WDMA, LIN>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, MAX_SMEM);
        });
        if (e != hipSuccess) return hip_result(e);
    }
    hipLaunchKernelGGL((bconv_mfma<TM, TN, WPH, WDMA, LIN>), dim3(blocks), dim3(256), smem, s, in, wt, g, ep);
    return hip_result(hipGetLastError());
}

template <int TM, int TN, int WPH, bool WDMA = false>
bnn_status launch_one(const uint32_t *in, const uint32_t *wt, int n, int h, int w, int c_in, int c_out,
                      const EpiArgs &ep, hipStream_t s)
{
    ConvGeom g;
    size_t smem;
    bool lin;
    if (pick_geom<TM, TN, WPH, WDMA>(n, h, w, c_in, c_out, ep.packed && ep.pool == 2, g, smem, &lin) < 0)
        return BNN_ERR_UNSUPPORTED;
    return lin ? launch_geom<TM, TN, WPH, WDMA, true>(in, wt, g, smem, ep, s)
               : launch_geom<TM, TN, WPH, WDMA, false>(in, wt, g, smem, ep, s);
}

// Estimated cost of a (64*TM pixels) x (64*TN channels) block tile, or a negative number if it does
// not fit LDS.  `items`: its work items (pixel tiles x channel tiles).  *lin: its tiles are linear.
template <int TM, int TN, int WPH, bool WDMA = false>
double cost_one(int n, int h, int w, int c_in, int c_out, bool win, bool *lin, int64_t *items = nullptr)
{
    ConvGeom g;
    size_t smem;
    const double cost = pick_geom<TM, TN, WPH, WDMA>(n, h, w, c_in, c_out, win, g, smem, lin);
    if (items) *items = cost < 0 ? 0 : (int64_t)g.n_ptiles * g.n_co_tiles;
    return cost;
}

}  // namespace

// The 256 x 128 tile of a channel width is compiled in a translation unit of its own (it is the
// slowest to build); the dispatcher below reaches it through this function.
template <int WPH>
bnn_status launch_conv_big_tile(const uint32_t *in, const uint32_t *wt, int n, int h, int w, int c_in,
                                int c_out, const EpiArgs &ep, hipStream_t s);

namespace {

// 64-channel tiles of 256 and 128 pixels, for channel counts that leave half of a 128-channel tile
// empty: weights resident, so up to twelve words per pixel.  (At two words the multiply phase is too
// short for them to matter.)
template <int WPH> constexpr bool narrow_tiles = WPH == 2 || WPH == 4 || WPH == 6;

// Which block tile launch_wph takes: the one of least estimated cost.  Over 219 layers (raw sums without the
// rule below) it takes 1.7 % more than the fastest tile and tiling on average and 5 % more for 26 of them;
// furthest off are layers that keep few MFMAs in flight (578 x 28 x 14, 384 -> 192 pooled 81 / 61 with 256 x 64, 1431 x 8 x 8, 192 -> 256
// 29.1 / 24.7 with 128 x 128).  The largest tile, which moves the least data, stays where it gives nearly
// every compute unit two blocks unless another promises 10 % less (without that 598 x 28 x 28, 64 -> 48
// 21.3 -> 27.1, 305 x 21 x 21, 448 -> 149 66.6 -> 80.3).
// us, largest / picked: 131 x 27 x 31, 256 -> 64 15.3 / 11.3 (256 x 64), 24 x 27 x 27, 400 -> 96
// 19.6 / 14.3 (128 x 128), 100 x 16 x 16, 320 -> 320 23.8 / 17.0 (256 x 64), 64 x 8 x 8, 512 -> 512
// 17.0 / 9.2 (64 x 64).
// 3: 256 x 128, 2: 128 x 128 with streamed weights, 1: 128 x 128, 4: 256 x 64, 5: 128 x 64,
// 0: 64 x 64.  win: a pooled layer (its tiles are made of 2x2 windows).  *raster: linear tiles.
// raw: raw sums alone.  They are mostly stores up to 256 channels, which the estimate leaves out and a block
// overlaps with another's multiplies only: smaller tiles.  us, with the largest tile allowed / without:
// 961 x 10 x 31, 64 -> 100 39.2 / 32.9, 941 x 15 x 15, 64 -> 155 145.4 / 129.7, 127 x 26 x 26, 64 -> 171
// 78.0 / 61.3, 589 x 31 x 31, 64 -> 56 47.4 / 39.9; 1.067 times as fast over 49 layers.  Slower are
// 450 x 20 x 20, 32 -> 188 39.3 / 41.4, 543 x 25 x 25, 128 -> 104 41.0 / 42.3, 192 x 18 x 18, 48 -> 372
// 25.0 / 25.7, 160 x 17 x 24, 160 -> 328 33.6 / 34.6.
template <int WPH>
int tile_choice_wph(int n, int h, int w, int c_in, int c_out, bool win, bool raw, bool *raster = nullptr)
{
    // the larger tiles keep their weights resident (WPH <= 4) or stream them by DMA
    constexpr bool WD = WPH >= 6;
    double best = -1;
    int choice = 0;
    bool lin = false, best_lin = false;
    auto take = [&](int c, double cost) {
        if (cost >= 0 && (best < 0 || cost < best)) { best = cost; choice = c; best_lin = lin; }
    };
    int64_t items;
    const double big = cost_one<4, 2, WPH, WD>(n, h, w, c_in, c_out, win, &lin, &items);
    if (!raw || WPH > 4) take(3, items >= 384 ? 0.9 * big : big);
    take(WD ? 2 : 1, cost_one<2, 2, WPH, WD>(n, h, w, c_in, c_out, win, &lin));
    if constexpr (narrow_tiles<WPH>) {
        take(4, cost_one<4, 1, WPH>(n, h, w, c_in, c_out, win, &lin));
        take(5, cost_one<2, 1, WPH>(n, h, w, c_in, c_out, win, &lin));
    }
    take(0, cost_one<1, 1, WPH>(n, h, w, c_in, c_out, win, &lin));
    if (raster) *raster = best_lin;
    return choice;
}

template <int WPH>
bnn_status launch_wph(const uint32_t *in, const uint32_t *wt, int n, int h, int w, int c_in, int c_out,
                      const EpiArgs &ep, hipStream_t s)
{
    constexpr bool WD = WPH >= 6;
    switch (tile_choice_wph<WPH>(n, h, w, c_in, c_out, ep.packed && ep.pool == 2, !ep.packed)) {
    case 3: return launch_conv_big_tile<WPH>(in, wt, n, h, w, c_in, c_out, ep, s);
    case 2:
    case 1: return launch_one<2, 2, WPH, WD>(in, wt, n, h, w, c_in, c_out, ep, s);
    case 4:
        if constexpr (narrow_tiles<WPH>) return launch_one<4, 1, WPH>(in, wt, n, h, w, c_in, c_out, ep, s);
        break;
    case 5:
        if constexpr (narrow_tiles<WPH>) return launch_one<2, 1, WPH>(in, wt, n, h, w, c_in, c_out, ep, s);
        break;
    }
    return launch_one<1, 1, WPH>(in, wt, n, h, w, c_in, c_out, ep, s);
}

}  // namespace

}  // namespace bnn
#endif
