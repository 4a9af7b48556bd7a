// Bandwidth-bound helpers for gfx950: bit packing of +-1 values, and the stand-alone
// step (+ 2x2 max-pool) layer on int32 pre-activations (paper Sec. II-A step / maxpool).
#include "bnn_internal.h"
#include "conv_epilogue.h"

namespace bnn {

namespace {

// 4 int8 in a dword -> 4 bits, bit q = (byte q > 0).
__device__ __forceinline__ unsigned positive_bits4(uint32_t w)
{
    // bit 7 of each byte: low 7 bits non-zero and sign bit clear
    const uint32_t m = (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) & ~w) & 0x80808080u;
    // gather bits 7,15,23,31 into bits 24..27 (distinct partial products, no carries)
    return (((m >> 7) * 0x01020408u) >> 24) & 0xfu;
}

__device__ __forceinline__ unsigned positive_bits16(const uint4 &v)
{
    return positive_bits4(v.x) | (positive_bits4(v.y) << 4) | (positive_bits4(v.z) << 8) |
           (positive_bits4(v.w) << 12);
}

// k % 32 == 0 and 16-byte aligned rows: one 16-byte load per lane, two lanes per word.
__global__ __launch_bounds__(256) void pack_bits_fast(const uint4 *__restrict__ src, int64_t n_half,
                                                      uint32_t *__restrict__ dst)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    // n_half is even and the loop trip count is wave-uniform up to the last partial wave;
    // lanes past the end compute zeros so that the pair shuffle stays convergent.
    for (int64_t base = (int64_t)blockIdx.x * 256; base < n_half; base += stride) {
        const int64_t i = base + threadIdx.x;
        unsigned bits = 0;
        if (i < n_half) bits = positive_bits16(src[i]);
        const unsigned other = __shfl_xor(bits, 1);
        if (i < n_half && (threadIdx.x & 1) == 0) dst[i >> 1] = bits | (other << 16);
    }
}

// 16 bytes at any byte address (the compiler may not assume more; the hardware takes it in one load).
__device__ __forceinline__ uint4 load16_unaligned(const void *p)
{
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// Any k: a row is 2 * kw half words of 16 source bytes, the last one or two of them short or empty;
// one 16-byte load per lane (at any byte address) and two lanes per word, as above.  Lanes follow
// the rows' bytes, so that a wave reads about 1 KB in one piece whatever k is.  A block takes
// HALVES consecutive half words: its first row is found with one division, a lane's row with a
// multiply-high.  (A tensor of fewer than 16 bytes goes to pack_bits_tiny.)  HBM-bound: 16384 x 5000 values 143 us with a thread per word and byte loads
// (0.65 TB/s), 16.0 us now (5.8 TB/s); 23804 x 773 42.6 / 5.9 us.
constexpr int PACK_UNROLL = 4, PACK_HALVES = 256 * PACK_UNROLL;

__global__ __launch_bounds__(256) void pack_bits_ragged(const int8_t *__restrict__ src, int64_t rows, int64_t k,
                                                        int64_t halves, unsigned mg, uint32_t *__restrict__ dst)
{
    const int64_t total = rows * halves;
    const int8_t *end = src + rows * k;
    for (int64_t base = (int64_t)blockIdx.x * PACK_HALVES; base < total; base += (int64_t)gridDim.x * PACK_HALVES) {
        const int64_t row0 = base / halves;
        const int64_t off0 = base - row0 * halves;
        const int8_t *p0 = src + row0 * k;
        uint4 v[PACK_UNROLL];
        int cnt[PACK_UNROLL], back[PACK_UNROLL];
#pragma unroll
        for (int u = 0; u < PACK_UNROLL; ++u) {
            const int64_t j = off0 + u * 256 + threadIdx.x;
            // (a block's span of a long row meets at most one more)
            const int r = halves >= PACK_HALVES ? (j >= halves ? 1 : 0) : div_by((int)j, (int)halves, mg);
            const int64_t at = (j - r * halves) * 16;                 // first byte inside the row
            const int8_t *p = p0 + r * k + at;
            const int64_t left = base + u * 256 + threadIdx.x < total ? k - at : 0;
            cnt[u] = left >= 16 ? 16 : (left > 0 ? (int)left : 0);
            // (a load that would pass the tensor's end reads its last 16 bytes, and `back` bytes of them
            // are shifted out below; a half word without bytes reads the same)
            const int8_t *lp = cnt[u] > 0 && end - p >= 16 ? p : end - 16;
            back[u] = cnt[u] > 0 ? (int)(p - lp) : 0;
            v[u] = load16_unaligned(lp);
        }
#pragma unroll
        for (int u = 0; u < PACK_UNROLL; ++u) {
            // (bytes behind the row's end belong to the next row)
            const unsigned bits = (positive_bits16(v[u]) >> back[u]) & ((1u << cnt[u]) - 1u);
            const unsigned other = __shfl_xor(bits, 1);
            const int64_t i = base + u * 256 + threadIdx.x;
            if (i < total && (threadIdx.x & 1) == 0) dst[i >> 1] = bits | (other << 16);
        }
    }
}

// Rows of at most 16 values: a lane per row and word, one 16-byte load (the rows' bytes overlap in the
// cache lines).  Two half words per row, as above, would leave every second lane without bytes: 1000003
// rows, us, a thread per word with byte loads / two half words / this: k = 2 3.84 / 7.74 / 3.86, k = 5 4.88 /
// 7.83 / 3.92, k = 15 10.4 / 8.0 / 4.56; single values stay with the byte load (10^7 rows 18.5, 22.2 with 16 bytes).
__global__ __launch_bounds__(256) void pack_bits_short(const int8_t *__restrict__ src, int64_t rows, int k,
                                                       uint32_t *__restrict__ dst)
{
    const int8_t *end = src + rows * k;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < rows; r += (int64_t)gridDim.x * 256) {
        const int8_t *p = src + r * k;
        if (k == 1) {
            dst[r] = *p > 0 ? 1u : 0u;
            continue;
        }
        const int8_t *lp = end - p >= 16 ? p : end - 16;         // (the tensor holds at least 16 bytes)
        dst[r] = (positive_bits16(load16_unaligned(lp)) >> (int)(p - lp)) & ((1u << k) - 1u);
    }
}

// At most 15 values in all: one thread.
__global__ void pack_bits_tiny(const int8_t *__restrict__ src, int rows, int k, uint32_t *__restrict__ dst)
{
    for (int r = 0; r < rows; ++r) {
        unsigned word = 0;
        for (int q = 0; q < k; ++q) word |= (src[r * k + q] > 0 ? 1u : 0u) << q;
        dst[r] = word;
    }
}

// Stand-alone step (+ pool).  A thread owns one group of eight channels, whose thresholds and flips
// it reads once, and walks over output pixels; four neighbouring lanes own a word.  A block's threads
// cover `gb` groups of 256 / gb pixels at a time, gb = min(groups per pixel, 256); the second grid index takes
// further groups (the grid is bx x by blocks in one dimension).  Output pixel p of a pooled layer is (q, x) with q = image and output row in one,
// and its window starts at input row 2q, column 2x: no other index is ever taken apart, and the step
// to the thread's next pixel is a fixed (q, x) increment.  HBM-bound.  Before, an item's four 64-bit
// divisions, eight flip bytes and eight thresholds were worked out and read anew for each pixel; us,
// before / after (at 6 TB/s): 256 x 32 x 32 x 128 77 / 22 (23), with pooling 35 / 20 (23);
// 1182 x 6 x 6 x 120 15.3 / 5.0 (3.5); 500 x 16 x 16 x 511 248 / 59 (45); 400 x 32 x 32 x 8 pooled 5.9 / 4.7 (2.2).
// Small layers are a chain of memory round trips, so no load waits for another's value: whole groups
// load without a branch, a short group's loads are guarded by its (uniform) size.
struct StepGeom {
    int64_t pixels;                  // output pixels
    int w, c, wo, cwo, gb;
    int pool_first;
    int64_t step_q;                  // a grid's worth of pixels as a (q, x) increment
    int step_x;
    int bx;
    unsigned mg_wo;                  // magic_floor of wo
};

// WHOLE: c is a multiple of eight, every group has eight channels or none.
template <int POOL, int U, bool WHOLE>                           // U: pixels of a thread in flight together
__global__ __launch_bounds__(256) void step_pool_kernel(const int32_t *__restrict__ x,
                                                        const int32_t *__restrict__ thr,
                                                        const uint8_t *__restrict__ flip, StepGeom g,
                                                        uint32_t *__restrict__ out)
{
    constexpr int WIN = POOL * POOL;
    static_assert(POOL == 1 || U == 1, "a pooled pixel has eight loads of its own");
    const int t = threadIdx.x, ppb = 256 / g.gb;
    const int slot = t / g.gb;
    const int yb = (int)blockIdx.x / g.bx, xb = (int)blockIdx.x - yb * g.bx;
    const int grp = yb * 256 + (t - slot * g.gb);
    if (slot >= ppb) return;                                     // (whole quads of lanes: gb is a multiple of 4)
    if (grp >= g.cwo * 4) return;                                // (whole quads again)
    const int nc = g.c - grp * 8 < 8 ? g.c - grp * 8 : 8;        // channels of the group that exist (may be <= 0)
    // (WHOLE: a group without channels reads the first one's and drops the result, no branch around its loads)
    const int c0 = WHOLE && nc <= 0 ? 0 : grp * 8;
    const int ns = g.c & 7;                                      // channels of the short group
    const unsigned valid = nc >= 8 ? 0xffu : (nc > 0 ? (1u << nc) - 1u : 0u);
    // thresholds and flips: three wide loads for a whole group (sixteen narrow gathers per thread made
    // the address unit the bound of small layers)
    int tv[8] = {};
    uint64_t fl = 0;                                             // flip bytes
    if (WHOLE || nc >= 8) {
        const int4 a = *reinterpret_cast<const int4 *>(thr + c0), b = *reinterpret_cast<const int4 *>(thr + c0 + 4);
        if (flip) __builtin_memcpy(&fl, flip + c0, 8);
        tv[0] = a.x; tv[1] = a.y; tv[2] = a.z; tv[3] = a.w;
        tv[4] = b.x; tv[5] = b.y; tv[6] = b.z; tv[7] = b.w;
    } else if (nc > 0) {
        uint8_t f[8] = {};
#pragma unroll
        for (int j = 0; j < 7; ++j)
            if (j < ns) {
                tv[j] = thr[c0 + j];
                if (flip) f[j] = flip[c0 + j];
            }
#pragma unroll
        for (int j = 0; j < 7; ++j) fl |= (uint64_t)f[j] << (8 * j);
    }
    int64_t p = (int64_t)xb * ppb + slot;
    const int64_t stride = (int64_t)g.bx * ppb;
    int64_t q = 0;
    int xo = 0;
    if (POOL == 2) {
        q = g.pixels < (int64_t)1 << 31 ? div_by((int)p, g.wo, g.mg_wo) : p / g.wo;
        xo = (int)(p - q * g.wo);
    }
    auto load8 = [&](const int32_t *src, int (&v)[8]) {
        if (WHOLE || nc >= 8) {
            const uint4 a = load16_unaligned(src), b = load16_unaligned(src + 4);
            v[0] = (int)a.x; v[1] = (int)a.y; v[2] = (int)a.z; v[3] = (int)a.w;
            v[4] = (int)b.x; v[5] = (int)b.y; v[6] = (int)b.z; v[7] = (int)b.w;
        } else if (nc > 0) {
#pragma unroll
            for (int j = 0; j < 7; ++j)
                if (j < ns) v[j] = src[j];
        }
    };
    unsigned fm = 0;                                             // flip bits
    auto step8 = [&](const int (&v)[8]) {
        unsigned b = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) b |= (v[j] > tv[j] ? 1u : 0u) << j;
        return b ^ fm;
    };
    for (; p < g.pixels; p += stride * U) {
        int v[U][WIN][8] = {};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (POOL == 1) {
                // (a pixel past the end reads the last one and is not stored)
                const int64_t pu = p + u * stride;
                load8(x + (pu < g.pixels ? pu : g.pixels - 1) * g.c + c0, v[u][0]);
            } else {
                const int32_t *src = x + (2 * q * g.w + 2 * xo) * g.c + c0;
                load8(src, v[u][0]);
                load8(src + g.c, v[u][1 % WIN]);
                load8(src + (int64_t)g.w * g.c, v[u][2 % WIN]);
                load8(src + (int64_t)(g.w + 1) * g.c, v[u][3 % WIN]);
            }
        }
        // (the flip bits are put together behind the pixels' loads, lest those wait for the flips)
        asm volatile("" : "+v"(fl));
        fm = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) fm |= ((fl >> (8 * j)) & 0xff ? 1u : 0u) << j;
        if (POOL == 2) {
            xo += g.step_x;
            q += g.step_q;
            if (xo >= g.wo) { xo -= g.wo; ++q; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            unsigned byte;
            if (POOL == 1) {
                byte = step8(v[u][0]);
            } else if (g.pool_first) {
                // paper order: max of the window's pre-activations, then the step
                int m[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    m[j] = max(max(v[u][0][j], v[u][1 % WIN][j]), max(v[u][2 % WIN][j], v[u][3 % WIN][j]));
                byte = step8(m);
            } else {
                byte = step8(v[u][0]) | step8(v[u][1 % WIN]) | step8(v[u][2 % WIN]) | step8(v[u][3 % WIN]);
            }
            unsigned word = (byte & valid) << (8 * (t & 3));
            word |= __shfl_xor(word, 1);
            word |= __shfl_xor(word, 2);
            const int64_t pu = p + u * stride;
            if (pu < g.pixels && (t & 3) == 0) out[pu * g.cwo + (grp >> 2)] = word;
        }
    }
}

unsigned grid_for(int64_t items)
{
    int64_t blocks = (items + 255) / 256;
    const int64_t cap = 256 * 32;     // 32 blocks per compute unit, grid-stride beyond
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (unsigned)blocks;
}

}  // namespace

bnn_status launch_pack_bits(const int8_t *src, int64_t rows, int64_t k, uint32_t *dst, hipStream_t s)
{
    if (rows == 0) return BNN_OK;
    const int64_t kw = (k + 31) / 32;
    if ((k & 31) == 0) {
        const int64_t n_half = rows * kw * 2;
        hipLaunchKernelGGL(pack_bits_fast, dim3(grid_for(n_half)), dim3(256), 0, s,
                           reinterpret_cast<const uint4 *>(src), n_half, dst);
    } else {
        if (rows * k < 16) {
            hipLaunchKernelGGL(pack_bits_tiny, dim3(1), dim3(1), 0, s, src, (int)rows, (int)k, dst);
            return hip_result(hipGetLastError());
        }
        if (k <= 16) {
            hipLaunchKernelGGL(pack_bits_short, dim3(grid_for(rows)), dim3(256), 0, s, src, rows, (int)k, dst);
            return hip_result(hipGetLastError());
        }
        const int64_t halves = 2 * kw;
        int64_t blocks = (rows * halves + PACK_HALVES - 1) / PACK_HALVES;
        if (blocks > 256 * 32) blocks = 256 * 32;
        hipLaunchKernelGGL(pack_bits_ragged, dim3((unsigned)blocks), dim3(256), 0, s, src, rows, k, halves,
                           halves < PACK_HALVES ? magic_floor((int)halves) : 0u, dst);
    }
    return hip_result(hipGetLastError());
}

bnn_status launch_threshold_sign_maxpool(const int32_t *x, int n, int h, int w, int c, const int32_t *thr,
                                         const uint8_t *flip, int pool, int pool_first, uint32_t *out,
                                         hipStream_t s)
{
    if (n == 0) return BNN_OK;
    StepGeom g;
    const int ho = h / pool;
    g.w = w; g.c = c; g.wo = w / pool; g.cwo = (c + 31) / 32; g.pool_first = pool_first;
    g.pixels = (int64_t)n * ho * g.wo;
    const int gpp = g.cwo * 4;
    g.gb = gpp < 256 ? gpp : 256;
    const int ppb = 256 / g.gb;
    // four pixels per thread in flight where that still leaves a block for every compute unit
    const bool four = pool == 1 && g.pixels >= (int64_t)ppb * 4 * 256;
    int64_t bx = (g.pixels + ppb * (four ? 4 : 1) - 1) / (ppb * (four ? 4 : 1));
    const int64_t by = (gpp + 255) / 256;
    const int64_t cap = by < 256 * 16 ? 256 * 16 / by : 1;      // blocks per compute unit, pixels strided beyond
    if (bx > cap) bx = cap;
    const int64_t stride = bx * ppb;
    g.step_q = stride / g.wo;
    g.step_x = (int)(stride - g.step_q * g.wo);
    g.bx = (int)bx;
    g.mg_wo = magic_floor(g.wo);
    const dim3 grid((unsigned)(bx * by));
#define BNN_STEP(POOL, U)                                                                                      \
    do {                                                                                                       \
        if ((c & 7) == 0) hipLaunchKernelGGL((step_pool_kernel<POOL, U, true>), grid, dim3(256), 0, s, x, thr, flip, g, out); \
        else hipLaunchKernelGGL((step_pool_kernel<POOL, U, false>), grid, dim3(256), 0, s, x, thr, flip, g, out); \
    } while (0)
    if (four) BNN_STEP(1, 4);
    else if (pool == 1) BNN_STEP(1, 1);
    else BNN_STEP(2, 1);
#undef BNN_STEP
    return hip_result(hipGetLastError());
}

}  // namespace bnn
