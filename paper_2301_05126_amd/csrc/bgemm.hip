// Binary fully-connected layer / binary GEMM for gfx950.
//
// C[r][o] = sum_t a[r][t] * b[o][t] over +-1 values stored one bit each
//         = 2*popcount(xnor) - #bits  (paper Sec. II-A neuron formula).
//
// Dense tiles run on the matrix cores: each 32-bit word of packed operand bits is expanded
// in registers into 32 FP4 (E2M1) values +-1.0 and fed to
// v_mfma_f32_32x32x64_f8f6f4 (the form without block scales).  Products are +-1 and partial sums are
// integers below 2^24, so the FP32 accumulators are exact.  Both operands use the same
// bit -> sign map (bit 1 -> -1.0) and the same permutation of K inside a word, neither of
// which changes a dot product.  Zero-filled words beyond K (and the zero tail bits of the
// last word) count as matches, a constant that the epilogue subtracts.
//
//   bgemm_mfma<TM,TN>  persistent blocks of 2x2 waves, wave tile (32*TM) x (32*TN), K streamed through
//                      LDS as packed words in chunks of 16 words, across the block's tiles.
//   bgemm_small        few 64 x 64 tiles: 32 x 32 outputs per block, K split over its four waves,
//                      operands straight from global memory.
//   bgemv_rows         m <= 8: bandwidth-bound, xor + popcount on the VALU, four output rows of
//                      B per wave, halving-butterfly reduction over the 64 lanes.
// All end in the same epilogue: optional int32 store, optional threshold/flip/bit-pack.  The two
// small-problem kernels can also carry the model's last layer (TAIL): each block adds the share
// of its 32-bit output words to the logits.
#include "bnn_internal.h"
#include "conv_epilogue.h"
#include "lds_dma.h"

namespace bnn {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Four words of a row without branches, so that many such loads can be in flight together: a
// word that does not exist reads the tensor's first word and is zeroed afterwards.
template <int VEC>
__device__ __forceinline__ uint4 load_row_words_nb(const uint32_t *__restrict__ base, int64_t row,
                                                   int64_t rows, int kw_total, int kpos)
{
    const bool row_ok = row < rows;
    const int64_t at = row * (int64_t)kw_total + kpos;
    uint4 v;
    if (VEC == 4) {
        const bool ok = row_ok && kpos < kw_total;
        v = *reinterpret_cast<const uint4 *>(base + (ok ? at : 0));
        v.x = ok ? v.x : 0u; v.y = ok ? v.y : 0u; v.z = ok ? v.z : 0u; v.w = ok ? v.w : 0u;
    } else if (VEC == 2) {
        const bool ok0 = row_ok && kpos < kw_total, ok1 = row_ok && kpos + 2 < kw_total;
        const uint2 lo = *reinterpret_cast<const uint2 *>(base + (ok0 ? at : 0));
        const uint2 hi = *reinterpret_cast<const uint2 *>(base + (ok1 ? at + 2 : 0));
        v = make_uint4(ok0 ? lo.x : 0u, ok0 ? lo.y : 0u, ok1 ? hi.x : 0u, ok1 ? hi.y : 0u);
    } else {
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool ok = row_ok && kpos + q < kw_total;
            const uint32_t x = base[ok ? at + q : 0];
            w[q] = ok ? x : 0u;
        }
        v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    return v;
}

__device__ __forceinline__ uint32_t word_of(const uint4 &v, int q)
{
    return q == 0 ? v.x : (q == 1 ? v.y : (q == 2 ? v.z : v.w));
}

// Makes a tile's accumulators opaque at this point, in the registers where they are: the compiler
// would otherwise copy them all out of the accumulation registers at the end of the loop, and spill.
__device__ __forceinline__ void pin_acc(v16f &acc) { asm volatile("" : "+a"(acc)); }

// Tiles of the problem.
struct GemmWalk {
    int nbm, nbn;            // tiles along M and N
    int tiles;               // nbm * nbn
    int stream;              // 1: streaming stores of raw sums
    int far;                 // raw sums: 32-bit offsets reach over a tile's rows (0), over eight rows (1), or not (2)
};

// Persistent blocks.  Tile numbers run column-major inside bands of eight tile rows; each XCD takes
// a contiguous eighth of them and its blocks (hardware deals block ids round-robin to the XCDs)
// walk through it side by side, so the tiles in flight on one L2 form a patch that shares rows of A
// and of B.
//
// K streams through four LDS buffers of KC = 16 words per row, filled by global -> LDS transfers
// that bypass the registers and are requested three chunks ahead.  A chunk costs one barrier, in its
// middle: there the next chunk is known to have landed for every wave and the previous one to be
// consumed, so the first words of the next chunk are read, and its first operands expanded, behind
// the last MFMAs of the current one.  The chunk sequence runs on across the block's tiles: the
// first chunks of the next tile are in flight during the last ones of this tile and during its
// epilogue, and the stores of a tile drain behind the first chunks of the next.
//
// What bounds it (256 x 256 tile): the MFMA pipe during the chunks, at 34.7 ticks per MFMA and SIMD of
// the 32 that a lone wave reaches with its operands in registers (46 with two barriers per chunk
// and staging through registers), and the power limit, which holds the clock at 1.9 GHz; then the
// stores of raw sums, 256 KB per tile and compute unit, in which the matrix pipe idles (9.4 us
// where all compute units store at once, the chip's write bandwidth; 5.7 us otherwise).  One block per
// tile with staging through registers / now, us: 16384^3 1518 / 1352, 8192^3 210 / 189, 4096^3 35.7 / 33.3 (a
// single round: 9 of its 33 us are the stores; kernel traces, two cards), step output at 5000 x 5000 x
// 10000 193 / 107, 4096 x 1024 x 8192 19.1 / 14.1.
//
// The smaller tiles expand two (64 x 64) or one (128 x 128) words per MFMA and are bound by the vector ALU,
// with one wave per SIMD also by what delays it: they make their operands from pairs of words, 5.5
// vector instructions per word instead of 7, and the next chunk's words are read one step behind
// the barrier (right behind it, a chunk took some 100 ticks longer at most alignments of the code).
// us, words one by one and read at the barrier / now: 896 x 896, K = 16384 17.2 / 15.0 (step output 16.4 /
// 14.3), 9 x 16384, K = 4096 6.1 / 5.6, 3000^3 21.8 / 20.8, 5000 x 5000, K = 1024 25.6 / 24.4.  Neither
// changes the 256 x 256 tile, and eight buffers instead of four make the 64 x 64 tile slower.
//
// An LDS row is four 16-byte units; unit u of row r sits at position u ^ ((r >> 1) & 3), so that the
// eight rows which one phase of a 16-byte read touches fall into distinct bank groups.  (A transfer
// writes 1 KB linearly; which unit a lane fetches makes the arrangement.)  Rows past M or N and
// words past K address past the end of the tile's buffer resource and arrive as zeros.
// VEC: 4 when rows are a whole number of 16-byte units, else 1 (four-byte transfers).
//
// B is the MFMA's first matrix: accumulator register r of lane (l32, half) is column 8(r/4) + 4*half +
// r%4 of a 32 x 32 tile and row l32, i.e. four neighbouring columns at a time: raw sums leave as
// 16-byte stores, and the step needs two instructions per value (see conv_epilogue.h).
constexpr int KC = 16, NBUF = 4, XW = 32 * 32;

// RAW / PACKED: which outputs the instance writes (one of the two in all but diagnostic calls).
// STORE: how raw sums leave.  QUADS: 16-byte stores; FAR: the same where rows are so long that 32-bit
// offsets do not reach over a tile's; LANES: 4-byte stores, a lane per column.
enum { QUADS = 0, FAR = 1, LANES = 2 };
template <int TM, int TN, int VEC, int OCC, bool RAW, bool PACKED, int STORE>
__global__ __launch_bounds__(256, OCC) void bgemm_mfma(const uint32_t *__restrict__ A,
                                                      const uint32_t *__restrict__ B, int64_t M, int64_t N,
                                                      int Kw, int K, GemmWalk gw, EpiArgs ep)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;     // 2 x 2 waves
    // operands made from pairs of words: the 256 x 256 tile has no registers to spare for it
    constexpr bool PAIR = TM * TN < 16;
    constexpr int IA = VEC == 4 ? TM : 4 * TM, IB = VEC == 4 ? TN : 4 * TN;   // transfers per wave and chunk
    constexpr int IPC = IA + IB;
    constexpr int ROWS_I = VEC == 4 ? 16 : 4;     // rows that one transfer fills
    constexpr int BUF = (BM + BN) * KC;           // words of one buffer: A's rows, then B's
    constexpr int NST = TM * TN * 4;              // 16-byte stores of a wave's tile
    constexpr int GJ = TM * TN >= 16 ? TN : 1;    // column tiles whose raw sums are stored together
    constexpr int AHEAD = NBUF - 1;               // chunks requested ahead
    constexpr int YOUNGER = (AHEAD - 2) * IPC;    // transfers younger than the chunk that is waited for
    static_assert(IPC <= 32, "the wait counter holds at most 63 transfers");
    extern __shared__ __align__(16) uint32_t smem[];

    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;
    // this wave's scratch of the epilogue: thresholds of its channels, or 32 x 32 sums
    float *Tw = reinterpret_cast<float *>(smem + NBUF * BUF) + wave * XW;
    int32_t *Xw = reinterpret_cast<int32_t *>(Tw);

    // ---- this block's tiles: numbers first, first + stride, ... of its XCD's share
    const int xcd = (int)blockIdx.x & 7, stride = (int)gridDim.x >> 3;
    const int x0 = (int)((int64_t)gw.tiles * xcd >> 3), x1 = (int)((int64_t)gw.tiles * (xcd + 1) >> 3);
    int tile = x0 + ((int)blockIdx.x >> 3);
    if (tile >= x1) return;
    auto origin = [&](int tl, int64_t &m0, int64_t &n0) {
        const int band = tl / (8 * gw.nbn);
        const int rows_in_band = min(8, gw.nbm - band * 8);
        const int idx = tl - band * 8 * gw.nbn;
        const int nb = idx / rows_in_band;
        m0 = (int64_t)(band * 8 + (idx - nb * rows_in_band)) * BM;
        n0 = (int64_t)nb * BN;
    };

    // ---- transfers.  Transfer j of this wave fills rows ROWS_I * (wave + 4 j) .. of A's (B's) part.
    const int nchunks = (Kw + KC - 1) / KC;
    const unsigned row_bytes = (unsigned)Kw * 4u;
    const int f_row = ROWS_I * wave + (VEC == 4 ? lane >> 2 : lane >> 4);
    const int f_unit = (VEC == 4 ? lane & 3 : (lane >> 2) & 3) ^ ((f_row >> 1) & 3);    // the same for every j
    const int f_word = f_unit * 4 + (VEC == 4 ? 0 : lane & 3);
    const unsigned f_off = (unsigned)f_row * row_bytes + (unsigned)f_word * 4u;
    const unsigned f_step = (unsigned)(4 * ROWS_I) * row_bytes;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) uint32_t *)smem +
                          (unsigned)wave * (ROWS_I * KC * 4);
    int tile_f = tile, c_f = 0, buf_f = 0;        // the chunk that is requested next, and its buffer
    v4i ra, rb;
    auto set_fetch_tile = [&]() {
        int64_t m0 = 0, n0 = 0;
        const bool on = tile_f < x1;
        if (on) origin(tile_f, m0, n0);
        // (past the block's last tile: an empty resource, every transfer delivers zeros, so that the
        // number of transfers in flight never depends on the tile)
        ra = make_raw_rsrc(A + m0 * Kw, on ? (unsigned)(M - m0 < BM ? M - m0 : BM) * row_bytes : 0u);
        rb = make_raw_rsrc(B + n0 * Kw, on ? (unsigned)(N - n0 < BN ? N - n0 : BN) * row_bytes : 0u);
    };
    // transfer j of the chunk (tile_f, c_f): A's first, then B's.  A word past K must not read the
    // next row: it addresses past the end of the resource instead.
    auto fetch = [&](int j) {
        const unsigned base = c_f * KC + f_word < Kw ? f_off + (unsigned)c_f * (KC * 4) : 0x80000000u;
        const bool is_a = j < IA;
        const int jj = is_a ? j : j - IA;
        const unsigned voff = base + (unsigned)jj * f_step;
        const unsigned at = lds0 + (unsigned)buf_f * (BUF * 4) + (unsigned)((is_a ? 0 : BM) + 4 * ROWS_I * jj) * (KC * 4);
        if (VEC == 4) lds_dma16(is_a ? ra : rb, at, voff);
        else lds_dma4(is_a ? ra : rb, at, voff);
    };
    auto fetch_next = [&]() {
        buf_f = buf_f + 1 == NBUF ? 0 : buf_f + 1;
        if (++c_f == nchunks) {
            c_f = 0;
            tile_f += stride;
            set_fetch_tile();
        }
    };
    set_fetch_tile();
#pragma unroll 1
    for (int c = 0; c < AHEAD; ++c) {
#pragma unroll
        for (int j = 0; j < IPC; ++j) fetch(j);
        fetch_next();
    }

    uint32_t sgn = 0x88888888u, one = 0x22222222u;
    asm volatile("" : "+s"(sgn));     // keep both masks in registers (v_and_or_b32 takes no literals)
    asm volatile("" : "+v"(one));

    // a chunk = two groups of 8 words; lane half h owns words [8g + 4h, 8g + 4h + 4) of group g,
    // i.e. unit 2g + h.  rd[g]: word offset of this lane's unit in a row of the wave's first tile.
    const int swz = ((l32 >> 1) & 3) ^ half;
    const int rd[2] = {l32 * KC + swz * 4, l32 * KC + (swz ^ 2) * 4};
    const int a0 = wm * TM * 32 * KC, b0 = (BM + wn * TN * 32) * KC;
    uint4 wa[2][TM], wb[2][TN];
    int buf = 0;                                              // buffer of the current chunk
    auto load_word = [&](int bf, int g, int w) {              // w: TM tiles of A, then TN of B
        const uint32_t *p = smem + bf * BUF + rd[g];
        if (w < TM) wa[g][w] = *reinterpret_cast<const uint4 *>(p + a0 + w * 32 * KC);
        else wb[g][w - TM] = *reinterpret_cast<const uint4 *>(p + b0 + (w - TM) * 32 * KC);
    };
    // transfers complete in order: with at most two younger chunks in flight the first has landed
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((AHEAD - 1) * IPC < 63 ? (AHEAD - 1) * IPC : IPC) : "memory");

#pragma unroll
    for (int w = 0; w < TM + TN; ++w) load_word(0, 0, w);

    const int corr = nchunks * KC * 32 - K;      // padded positions all counted as +1
    int after_stores = 0;                        // 1: the previous tile's epilogue was exactly NST stores

#pragma unroll 1
    for (; tile < x1; tile += stride) {
        int64_t m0, n0;
        origin(tile, m0, n0);
        // thresholds and flips of this wave's channels, one or two per lane, needed after the sums
        int thr[(TN + 1) / 2];
        unsigned flip[(TN + 1) / 2];
        if (PACKED) {
#pragma unroll
            for (int q = 0; q < (TN + 1) / 2; ++q) {
                const int64_t col = n0 + wn * TN * 32 + q * 64 + lane;
                const int64_t cl = col < N ? col : N - 1;
                thr[q] = ep.thr[cl];
                flip[q] = ep.flip && col < N ? ep.flip[cl] : 0u;
            }
        }
        // (opaque, so that the start value is not kept in registers of its own across the tiles)
        float start = -(float)corr;
        asm volatile("" : "+v"(start));
        v16f acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = start;

        // operands of the current and the next step (FP4: the low four dwords of an MFMA operand)
        v4i a[2][TM], b[2][TN];
        auto operand = [](const v4i &x) { return v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0}; };
        // words 2p and 2p + 1 of a group: the words of two consecutive steps (see shift_pair_half)
        auto pair_of = [](const uint4 &v, int p) { return p == 0 ? make_uint2(v.x, v.y) : make_uint2(v.z, v.w); };
        auto expand4 = [&](const uint4 &v) {
            if (!PAIR) {
                const v8i e = expand_fp4(v.x, sgn, one);
                return v4i{e[0], e[1], e[2], e[3]};
            }
            const uint2 lo = expand_pair_half(pair_of(v, 0), 0, 0, sgn, one), hi = expand_pair_half(pair_of(v, 0), 0, 1, sgn, one);
            return v4i{(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
        };
#pragma unroll
        for (int i = 0; i < TM; ++i) a[0][i] = expand4(wa[0][i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[0][j] = expand4(wb[0][j]);

        constexpr int NM = TM * TN, NW = TM + TN;
#pragma unroll 1
        for (int c = 0;;) {
            const int lax = __builtin_amdgcn_readfirstlane(after_stores & (c < AHEAD - 1 ? 1 : 0));
            const int buf_n = buf + 1 == NBUF ? 0 : buf + 1;
            // The order below is the issue order (scheduling barriers pin it): each MFMA is followed by
            // its share of the LDS reads, transfers and next step's operand dwords.
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                const int cur = st & 1, nxt = cur ^ 1;
                const int g1 = ((st + 1) >> 2) & 1, q1 = (st + 1) & 3;
                // The next chunk has landed and every wave is past the previous one, whose buffer takes
                // the chunk after the next two.  One younger chunk may be in flight; in a tile's first
                // two chunks also the previous tile's stores, which are younger than the chunk waited for.
                if (st == 4)
                    asm volatile("s_waitcnt vmcnt(%0)\n\t"
                                 "s_cmp_lg_u32 %2, 0\n\t"
                                 "s_cbranch_scc1 .Lgemm_lax%=\n\t"
                                 "s_waitcnt vmcnt(%1)\n"
                                 ".Lgemm_lax%=:\n\t"
                                 "s_barrier" ::"n"(YOUNGER + NST < 63 ? YOUNGER + NST : 63), "n"(YOUNGER), "s"(lax) : "memory", "scc");
                uint2 pend[2 * NW];                       // shifted pairs awaiting their masks
#pragma unroll
                for (int k = 0; k < NM; ++k) {
                    const int i = k / TN, j = k % TN;
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(b[cur][j]), operand(a[cur][i]),
                                                                                acc[i][j], 4, 4, 0, 0, 0, 0);
                    if (st == 0 || st == 5) {              // this chunk's second group, the next one's first
#pragma unroll
                        for (int w = k * NW / NM; w < (k + 1) * NW / NM; ++w)
                            load_word(st == 0 ? buf : buf_n, st == 0 ? 1 : 0, w);
                    }
                    if (st == 6) {
#pragma unroll
                        for (int f = k * IPC / NM; f < (k + 1) * IPC / NM; ++f) fetch(f);
                    }
                    if constexpr (PAIR) {
                        // the next step's operands, two dwords at a time: a shift of a pair of words, and one
                        // MFMA later (LAG) its masks, so that no instruction waits for the one before it
                        constexpr int NIT = 2 * NW, LAG = NM > 1 ? 1 : 0;
#pragma unroll
                        for (int t2 = 0; t2 < NIT; ++t2) {
                            const int ks = t2 * (NM - LAG) / NIT;           // the MFMA that the shift follows
                            const int w = t2 >> 1, dp = t2 & 1;
                            if (ks == k) pend[t2] = shift_pair_half(pair_of(w < TM ? wa[g1][w] : wb[g1][w - TM], q1 >> 1), q1 & 1, dp);
                            if (ks + LAG == k) {
                                const uint2 e = mask_pair(pend[t2], sgn, one);
                                v4i &o = w < TM ? a[nxt][w] : b[nxt][w - TM];
                                o[2 * dp] = (int)e.x;
                                o[2 * dp + 1] = (int)e.y;
                                // (used here, lest the next chunk's first operands be made after the last MFMA)
                                if (st == 7 && dp == 1) asm volatile("" ::"v"(o));
                            }
                        }
                    } else {
#pragma unroll
                        for (int d = k * 4 * NW / NM; d < (k + 1) * 4 * NW / NM; ++d) {
                            const int w = d >> 2, part = d & 3;
                            if (w < TM) a[nxt][w][part] = (int)expand_part(word_of(wa[g1][w], q1), part, sgn, one);
                            else b[nxt][w - TM][part] = (int)expand_part(word_of(wb[g1][w - TM], q1), part, sgn, one);
                            // (used here, lest the next chunk's first operands be made after the last MFMA)
                            if (st == 7 && part == 3) asm volatile("" ::"v"(w < TM ? a[nxt][w] : b[nxt][w - TM]));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            buf = buf_n;
            fetch_next();
            if (++c == nchunks) break;
        }

        // ---- epilogue: register r of lane (l32, half) in tile (i, j) is row 32i + l32 of the wave's part,
        // column 32j + 8(r/4) + 4*half + r%4
        const int row0 = wm * TM * 32 + l32, col0 = wn * TN * 32;
        const int rows = (int)(M - m0 < BM ? M - m0 : BM);
        after_stores = 0;
        if constexpr (RAW) {
            // One 32 x 32 tile after the other through the wave's own LDS area, so that a store covers
            // eight rows of 128 contiguous bytes: a lane writes its row's four quads of columns (quad c of
            // row r at position c ^ (r % 8): no bank conflicts either way) and reads quad lane % 8 of
            // rows lane / 8 + 8k.  Whole cache lines matter: quads stored as they come out of the
            // accumulators (32 bytes to a row) take 308 us at 8192^3, 64 bytes to a row 212 us, 128
            // bytes 195 us, and the 512 that the 256 x 256 tile writes in one go 193 us.  The stores go
            // through a buffer resource over the tile's rows of C, or (FAR) over eight of them at a time: a
            // row past M or a column past N addresses past its end and is dropped.
            // Where not even eight rows fit, 64-bit addresses.  LANES: a small tile that is its block's only
            // one, of a C whose rows are no whole number of quads: its stores are not hidden behind another
            // tile's chunks, and quads on 4-byte addresses drain slowly (2500 x 2501, K = 1000 10.75 us with
            // quads, 10.18 so; 2000 x 2001, K = 300 9.33 / 8.64; 1500 x 1501, K = 300 7.23 / 7.28).  (Instances of
            // their own: eight rows at a time always takes up to 7 % longer, and a branch more in the
            // epilogue cost the smallest products 3 %.)
            const unsigned c_row = (unsigned)N * 4u;
            const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(
                ep.preact + m0 * N, 0, (int)((unsigned)rows * c_row), 0x00020000);
            const int sr = lane >> 3, sq = lane & 7;
            int32_t *wr[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) wr[q] = Xw + l32 * 32 + (((2 * q + half) ^ (l32 & 7)) << 2);
            const int32_t *rp = Xw + sr * 32 + ((sq ^ sr) << 2);
            const unsigned col = (unsigned)(n0 + col0) + sq * 4u;            // of tile column 0
            unsigned at = (unsigned)(wm * TM * 32 + sr) * c_row + col * 4u;
            const bool whole = (N & 3) == 0 || n0 + BN <= N;                // a quad is all inside or all outside
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int j0 = 0; j0 < TN; j0 += GJ) {
                    v4i x[GJ][4];                  // a row's GJ * 128 bytes leave one after the other
#pragma unroll
                    for (int j = 0; j < GJ; ++j) {
                        v16f &ac = acc[i][j0 + j];
                        if (!PACKED) pin_acc(ac);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<int4 *>(wr[q]) =
                                make_int4((int)ac[q * 4], (int)ac[q * 4 + 1], (int)ac[q * 4 + 2], (int)ac[q * 4 + 3]);
                        // (other lanes of the wave read what this one wrote: LDS keeps a wave's order)
                        asm volatile("" ::: "memory");
#pragma unroll
                        for (int k = 0; k < 4; ++k) x[j][k] = *reinterpret_cast<const v4i *>(rp + k * 256);
                        asm volatile("" ::: "memory");
                        __builtin_amdgcn_sched_barrier(0);      // one tile's registers at a time
                    }
                    const int r0 = wm * TM * 32 + i * 32;
                    if constexpr (STORE == FAR) {
                        if (gw.far == 1) {
                            const unsigned at8 = (unsigned)sr * c_row + col * 4u;
                            auto rows8 = [&](int k) {
                                const int left = rows - (r0 + 8 * k);
                                return __builtin_amdgcn_make_buffer_rsrc(
                                    ep.preact + (m0 + r0 + 8 * k) * N, 0,
                                    (int)((unsigned)(left < 0 ? 0 : (left < 8 ? left : 8)) * c_row), 0x00020000);
                            };
                            if (whole) {
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const __amdgpu_buffer_rsrc_t c8 = rows8(k);
#pragma unroll
                                    for (int j = 0; j < GJ; ++j) {
                                        const int jj = j0 + j;
                                        const unsigned aj = col + jj * 32 < (unsigned)N ? at8 + jj * 128 : 0x80000000u;
                                        if (gw.stream) __builtin_amdgcn_raw_buffer_store_b128(x[j][k], c8, aj, 0, 2);
                                        else __builtin_amdgcn_raw_buffer_store_b128(x[j][k], c8, aj, 0, 0);
                                    }
                                }
                            } else {
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const __amdgpu_buffer_rsrc_t c8 = rows8(k);
#pragma unroll
                                    for (int j = 0; j < GJ; ++j)
#pragma unroll
                                        for (int e = 0; e < 4; ++e) {
                                            const int jj = j0 + j;
                                            const unsigned ae =
                                                col + jj * 32 + e < (unsigned)N ? at8 + (jj * 128 + e * 4) : 0x80000000u;
                                            __builtin_amdgcn_raw_buffer_store_b32(x[j][k][e], c8, ae, 0, 0);
                                        }
                                }
                            }
                        } else {
                            int32_t *cp = ep.preact + (m0 + r0 + sr) * N + n0 + col0 + j0 * 32 + sq * 4;
#pragma unroll
                            for (int k = 0; k < 4; ++k, cp += 8 * N)
#pragma unroll
                                for (int j = 0; j < GJ; ++j) {
                                    const int64_t left = r0 + sr + k * 8 < rows ? N - (n0 + col0 + (j0 + j) * 32 + sq * 4) : 0;
                                    if (left >= 4 && (N & 3) == 0) {
                                        *reinterpret_cast<v4i *>(cp + j * 32) = x[j][k];
                                    } else {
#pragma unroll
                                        for (int e = 0; e < 4; ++e)
                                            if (e < left) cp[j * 32 + e] = x[j][k][e];
                                    }
                                }
                        }
                    } else if constexpr (STORE == LANES) {
                        const unsigned cl = (unsigned)(n0 + col0) + j0 * 32 + l32;
                        const unsigned al = (unsigned)(r0 + half) * c_row + cl * 4u;
#pragma unroll
                        for (int k = 0; k < 16; ++k) {                    // rows 2k and 2k + 1, a lane per column
                            const int row = 2 * k + half;
                            const int v = Xw[row * 32 + (((l32 >> 2) ^ (row & 7)) << 2) + (l32 & 3)];
                            __builtin_amdgcn_raw_buffer_store_b32(v, crs, (cl < (unsigned)N ? al : 0x80000000u) + 2 * k * c_row, 0, 0);
                        }
                        asm volatile("" ::: "memory");
                    } else if (whole) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int j = 0; j < GJ; ++j) {
                                const int jj = j0 + j;
                                const unsigned aj = (col + jj * 32 < (unsigned)N ? at + jj * 128 : 0x80000000u) + k * 8 * c_row;
                                if (gw.stream) __builtin_amdgcn_raw_buffer_store_b128(x[j][k], crs, aj, 0, 2);
                                else __builtin_amdgcn_raw_buffer_store_b128(x[j][k], crs, aj, 0, 0);
                            }
                    } else {
#pragma unroll
                        for (int j = 0; j < GJ; ++j)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int jj = j0 + j;
                                const unsigned ae = col + jj * 32 + e < (unsigned)N ? at + (jj * 128 + e * 4) : 0x80000000u;
#pragma unroll
                                for (int k = 0; k < 4; ++k)
                                    __builtin_amdgcn_raw_buffer_store_b32(x[j][k][e], crs, ae + k * 8 * c_row, 0, 0);
                            }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                at += 32 * c_row;
            }
            after_stores = whole && !PACKED && STORE != LANES && (STORE != FAR || gw.far == 1);
        }
        if constexpr (PACKED) {
            // thresholds through LDS (written and read by the same wave) into the accumulators' channel
            // order; T - x is negative iff x > T (both exact, a difference never rounds to zero)
            unsigned flipw[TN];
#pragma unroll
            for (int q = 0; q < (TN + 1) / 2; ++q) {
                const int bound = K + 1;                      // no sum reaches it
                const int th = thr[q] > bound ? bound : (thr[q] < -bound ? -bound : thr[q]);
                if (q * 64 + lane < TN * 32) Tw[q * 64 + lane] = (float)th;
                const unsigned long long fl = __ballot(flip[q] != 0);
                flipw[2 * q] = (unsigned)fl;
                if (2 * q + 1 < TN) flipw[2 * q + 1] = (unsigned)(fl >> 32);
            }
            asm volatile("" ::: "memory");
            const int64_t nw = (N + 31) >> 5, w0 = (n0 + col0) >> 5;
            auto okw = [&](int j) {                           // channels of tile j that exist
                const int64_t left = N - (n0 + col0 + j * 32);
                return left >= 32 ? 0xffffffffu : (left <= 0 ? 0u : (1u << left) - 1u);
            };
            constexpr int JS = TN % 2 == 0 ? 2 : 1;
#pragma unroll
            for (int jp = 0; jp < TN; jp += JS) {
                v16f tv[JS];
#pragma unroll
                for (int u = 0; u < JS; ++u) tv[u] = load_bias16<v16f>(Tw + (jp + u) * 32, half);
                unsigned fl = flipw[jp], ok = okw(jp);
                if (JS == 2) {
                    fl = half ? flipw[jp + JS - 1] : fl;
                    ok = half ? okw(jp + JS - 1) : ok;
                }
                const int64_t wi = w0 + jp + (JS == 2 ? half : 0);
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    if (!RAW) pin_acc(acc[i][jp]);
                    if (!RAW && JS == 2) pin_acc(acc[i][jp + JS - 1]);
                    const unsigned lo = tile_half_word<false>([&](int r) { return tv[0][r] - acc[i][jp][r]; });
                    const unsigned hi =
                        JS == 2 ? tile_half_word<false>([&](int r) { return tv[JS - 1][r] - acc[i][jp + JS - 1][r]; }) : lo;
                    // two tiles' words: the first complete in lanes 0..31, the second in lanes 32..63
                    const auto sw = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
                    const unsigned word = (merge_half_words(sw[0], sw[1]) ^ fl) & ok;
                    if (row0 + i * 32 < rows && wi < nw && (JS == 2 || half == 0))
                        ep.packed[(m0 + row0 + i * 32) * nw + wi] = word;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    // nothing may be on its way to LDS when the block gives it back
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Small dense problems (the 64 x 64 tiling would leave most compute units idle): a block owns
// 32 x 32 outputs and its four waves split K in units of four MFMA steps (eight packed words per
// row; lane half h owns words [8u + 4h, 8u + 4h + 4) of unit u, one 16-byte load per operand, lane
// and unit).  Wave v takes the units v, v + 4, ... in rounds of up to eight units with all loads
// of a round in flight together, straight from global memory (no staging, no barrier before the
// MFMAs); the partial sums meet in LDS, and each wave adds up and finishes eight of the 32 rows.
// Latency, not throughput: with a quarter of K per wave and four times the blocks, a batch-256 FC
// layer of K = 8192 takes half the time of the 64 x 64 tile.  The block's last part is a serial chain,
// so it is split: wave 0 alone, with thresholds fetched after the sums, took 0.8 us more (device us,
// before / after: 64 x 512, K = 512 3.6 / 2.9; 256 x 1024, K = 8192 6.1 / 5.4).
//
// TAIL (see bgemv_rows): the block's 32 output words, one per row, each give their share of at
// most 16 logits per row; thread t adds those of row t % 32 and classes t / 32 and t / 32 + 8.
template <int VEC, bool TAIL>
__global__ __launch_bounds__(256) void bgemm_small(const uint32_t *__restrict__ A, const uint32_t *__restrict__ B,
                                                   int64_t M, int64_t N, int Kw, int K, int nbn, EpiArgs ep,
                                                   FcTailArgs tail)
{
    constexpr int UR = 8;                   // units per wave and round
    __shared__ v4f red[4][4][64];           // partial sums: [wave][four registers][lane]
    __shared__ uint32_t out_word[32];
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int64_t m0 = (int64_t)(blockIdx.x / nbn) * 32;
    const int64_t n0 = (int64_t)(blockIdx.x % nbn) * 32;
    const int units = (Kw + 7) >> 3;

    uint32_t w_tail[2] = {0u, 0u};          // on their way while the dot products run
    if (TAIL) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int j = (t >> 5) + 8 * i;
            if (j < tail.n_out) w_tail[i] = tail.w[(int64_t)j * ((N + 31) >> 5) + (n0 >> 5)];
        }
    }
    const int64_t col = n0 + l32;
    const bool cok = col < N;
    int thr = 0;                            // (these too)
    unsigned flipv = 0;
    if (ep.packed) {
        thr = ep.thr[cok ? col : 0];
        if (ep.flip) flipv = ep.flip[cok ? col : 0];
    }

    uint32_t sgn = 0x88888888u, one = 0x22222222u;
    asm volatile("" : "+s"(sgn));
    asm volatile("" : "+v"(one));
    v16f acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    for (int u0 = wave; u0 < units; u0 += 4 * UR) {
        uint4 wa[UR], wb[UR];
#pragma unroll
        for (int k = 0; k < UR; ++k) {
            const int u = u0 + 4 * k;
            // (a unit or a row past the end gives zeros)
            wa[k] = load_row_words_nb<VEC>(A, m0 + l32, M, Kw, u * 8 + half * 4);
            wb[k] = load_row_words_nb<VEC>(B, n0 + l32, N, Kw, u * 8 + half * 4);
        }
#pragma unroll
        for (int k = 0; k < UR; ++k) {
            if (u0 + 4 * k < units) {       // uniform per wave
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        expand_fp4(word_of(wa[k], q), sgn, one), expand_fp4(word_of(wb[k], q), sgn, one), acc, 4, 4,
                        0, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) red[wave][q][lane] = v4f{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    __syncthreads();
    {
        // register r of lane (l32, half) is row 8(r/4) + 4*half + r%4, column l32; this wave's are the
        // registers 4 * wave .. 4 * wave + 3 (small integers: exact in any order)
        v4f sum = red[0][wave][lane];
#pragma unroll
        for (int v = 1; v < 4; ++v) sum += red[v][wave][lane];
        const int corr = units * 8 * 32 - K;        // zero words and tail bits all counted as +1
        const int r0 = wave * 8 + half * 4;
        if (ep.preact) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (m0 + r0 + i < M && cok) ep.preact[(m0 + r0 + i) * N + col] = (int)sum[i] - corr;
        }
        if (ep.packed) {
            const int64_t nw = (N + 31) >> 5;
            unsigned mine = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int x = (int)sum[i] - corr;
                const unsigned long long mask = __ballot(cok && ((x > thr) != (flipv != 0)));
                const unsigned word = half ? (unsigned)(mask >> 32) : (unsigned)mask;
                if (l32 == i) mine = word;          // lane i of each half keeps the word of its row i
            }
            if (l32 < 4 && m0 + r0 + l32 < M) ep.packed[(m0 + r0 + l32) * nw + (n0 >> 5)] = mine;
            if (TAIL && l32 < 4) out_word[r0 + l32] = mine;
        }
    }
    if (TAIL) {
        __syncthreads();
        const int r = t & 31;
        const int64_t left = N - n0;                        // output bits the block's words hold
        const int valid = left < 32 ? (int)left : 32;
        const uint32_t mask = valid < 32 ? ((1u << valid) - 1u) : 0xffffffffu;
        const uint32_t wd = out_word[r];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int j = (t >> 5) + 8 * i;
            if (j < tail.n_out && m0 + r < M)
                atomicAdd(&tail.logits[(m0 + r) * tail.n_out + j],
                          valid - 2 * __builtin_popcount((wd ^ w_tail[i]) & mask));
        }
    }
}

// m <= MT rows of A (batch 1 .. 8): bandwidth / latency bound, on the VALU.
// Block = 8 waves = 32 consecutive outputs (one packed word); wave w owns outputs 4w..4w+3
// and streams their B rows with all loads of a K slice in flight at once.  Lanes stride K
// (16 bytes per lane when VEC == 4), accumulate popcount(a ^ b), then a halving butterfly
// reduces the 4 partial sums per lane over the 64 lanes with 2 + 1 + 4 shuffles per row.
//
// TAIL: the layer after this one is the model's last, which has no step and is therefore linear
// in this layer's output bits.  A block holds one whole 32-bit word of every output row, so it
// adds that word's share of each logit, valid - 2 popcount((word ^ w) & mask), to the logits with
// integer atomics (exact and independent of the order of arrival); the logits must be zero when
// the launch starts.  One thread per (row, logit): M * n_out <= 512.
template <int MT, int VEC, bool TAIL>
__global__ __launch_bounds__(512) void bgemv_rows(const uint32_t *__restrict__ A,
                                                  const uint32_t *__restrict__ B, int M, int64_t N, int Kw,
                                                  int K, EpiArgs ep, FcTailArgs tail)
{
    __shared__ int xs[MT][32];
    __shared__ uint32_t out_word[MT];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t o_base = (int64_t)blockIdx.x * 32;

    // this thread's word of the last layer's weights, on its way while the dot products run
    uint32_t w_tail = 0;
    int tail_r = 0, tail_j = 0;
    const bool tail_on = TAIL && (int)threadIdx.x < M * tail.n_out;
    if (tail_on) {
        tail_r = (int)threadIdx.x / tail.n_out;
        tail_j = (int)threadIdx.x - tail_r * tail.n_out;
        w_tail = tail.w[(int64_t)tail_j * ((N + 31) >> 5) + blockIdx.x];
    }

    int acc[MT][4];
#pragma unroll
    for (int r = 0; r < MT; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[r][q] = 0;

    const uint32_t *brow[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t o = o_base + wave * 4 + q;
        brow[q] = B + (o < N ? o : N - 1) * (int64_t)Kw;      // rows past N are computed, never stored
    }
    if (VEC == 4) {
        for (int kb = lane * 4; kb < Kw; kb += 256) {
            uint4 b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = *reinterpret_cast<const uint4 *>(brow[q] + kb);
#pragma unroll
            for (int r = 0; r < MT; ++r) {
                if (r < M) {
                    const uint4 a = *reinterpret_cast<const uint4 *>(A + (int64_t)r * Kw + kb);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[r][q] += __builtin_popcount(a.x ^ b[q].x) + __builtin_popcount(a.y ^ b[q].y) +
                                     __builtin_popcount(a.z ^ b[q].z) + __builtin_popcount(a.w ^ b[q].w);
                }
            }
        }
    } else {
        for (int kb = lane; kb < Kw; kb += 64) {
            uint32_t b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = brow[q][kb];
#pragma unroll
            for (int r = 0; r < MT; ++r) {
                if (r < M) {
                    const uint32_t a = A[(int64_t)r * Kw + kb];
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[r][q] += __builtin_popcount(a ^ b[q]);
                }
            }
        }
    }

    // halving butterfly: after the exchanges with lane^32 and lane^16 a lane keeps the sum of
    // output q = 2*bit5 + bit4; the remaining four exchanges finish the sum over 16 lanes.
#pragma unroll
    for (int r = 0; r < MT; ++r) {
        if (r >= M) break;
        const bool hi5 = (lane & 32) != 0, hi4 = (lane & 16) != 0;
        const int s0 = hi5 ? acc[r][0] : acc[r][2], s1 = hi5 ? acc[r][1] : acc[r][3];   // what the partner keeps
        const int k0 = hi5 ? acc[r][2] : acc[r][0], k1 = hi5 ? acc[r][3] : acc[r][1];   // what this lane keeps
        const int t0 = k0 + __shfl_xor(s0, 32), t1 = k1 + __shfl_xor(s1, 32);
        int v = (hi4 ? t1 : t0) + __shfl_xor(hi4 ? t0 : t1, 16);
        v += __shfl_xor(v, 8);
        v += __shfl_xor(v, 4);
        v += __shfl_xor(v, 2);
        v += __shfl_xor(v, 1);
        if ((lane & 15) == 0) xs[r][wave * 4 + (lane >> 4)] = K - 2 * v;
    }
    __syncthreads();

    const int tid = threadIdx.x;
    if (tid < 256) {                // 8 rows x 32 outputs; waves 0..3 are entirely inside
        const int r = tid >> 5;
        const int ol = tid & 31;
        const int64_t o = o_base + ol;
        const bool ok = (r < MT) && (r < M) && (o < N);
        const int x = ok ? xs[r < MT ? r : 0][ol] : 0;
        if (ep.preact && ok) ep.preact[(int64_t)r * N + o] = x;
        if (ep.packed) {
            bool bit = false;
            if (ok) {
                bit = x > ep.thr[o];
                if (ep.flip && ep.flip[o]) bit = !bit;
            }
            const unsigned long long mask = __ballot(bit);   // lanes 0-31: row r, 32-63: row r+1
            const unsigned word = (lane < 32) ? (unsigned)(mask & 0xffffffffull) : (unsigned)(mask >> 32);
            const int64_t nw = (N + 31) >> 5;
            if (ol == 0 && r < M && r < MT) {
                ep.packed[(int64_t)r * nw + blockIdx.x] = word;
                if (TAIL) out_word[r] = word;
            }
        }
    }
    if (TAIL) {
        __syncthreads();
        if (tail_on) {
            const int64_t left = N - o_base;                 // output bits this block's word holds
            const int valid = left < 32 ? (int)left : 32;
            const uint32_t mask = valid < 32 ? ((1u << valid) - 1u) : 0xffffffffu;
            const int part = valid - 2 * __builtin_popcount((out_word[tail_r] ^ w_tail) & mask);
            atomicAdd(&tail.logits[(int64_t)tail_r * tail.n_out + tail_j], part);
        }
    }
}

template <int TM, int TN, int VEC, bool RAW, bool PACKED, int STORE = QUADS>
bnn_status launch_mfma_out(const uint32_t *a, int64_t m, int64_t k, const uint32_t *b, int64_t n, int kw,
                           const GemmWalk &gw, const EpiArgs &ep, hipStream_t s)
{
    // blocks per compute unit: the 256 x 256 tile fills the registers, the smaller ones the LDS
    constexpr int OCC = TM * TN >= 16 ? 1 : 2;
    constexpr int RES = TM * TN >= 16 ? 1 : (TM * TN >= 4 ? 2 : 3);
    if constexpr (RAW && STORE == QUADS) {
        if (gw.far) return launch_mfma_out<TM, TN, VEC, RAW, PACKED, FAR>(a, m, k, b, n, kw, gw, ep, s);
        if constexpr (TM * TN < 16 && !PACKED) {
            if ((n & 3) != 0 && gw.tiles <= 256 * RES)
                return launch_mfma_out<TM, TN, VEC, RAW, PACKED, LANES>(a, m, k, b, n, kw, gw, ep, s);
        }
    }
    constexpr unsigned smem = (NBUF * 64 * (TM + TN) * KC + 4 * XW) * 4;
    static_assert(RES * smem <= 160 * 1024, "LDS of the resident blocks");
    if (smem > 64 * 1024) {          // above the default limit of dynamic LDS: opt in, once per kernel and device
        static PerDevice raised;
        const hipError_t e = raised.run([] {
            return hipFuncSetAttribute((const void *)bgemm_mfma<TM, TN, VEC, OCC, RAW, PACKED, STORE>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        });
        if (e != hipSuccess) return hip_result(e);
    }
    // a whole number of blocks per XCD; those without a tile leave at once
    const unsigned blocks = 8u * (unsigned)ceil_div64(gw.tiles < 256 * RES ? gw.tiles : 256 * RES, 8);
    hipLaunchKernelGGL((bgemm_mfma<TM, TN, VEC, OCC, RAW, PACKED, STORE>), dim3(blocks), dim3(256), smem, s, a, b, m, n, kw,
                       (int)k, gw, ep);
    return hip_result(hipGetLastError());
}

template <int TM, int TN, int VEC>
bnn_status launch_mfma_vec(const uint32_t *a, int64_t m, int64_t k, const uint32_t *b, int64_t n, int kw,
                           const GemmWalk &gw, const EpiArgs &ep, hipStream_t s)
{
    if (!ep.packed) return launch_mfma_out<TM, TN, VEC, true, false>(a, m, k, b, n, kw, gw, ep, s);
    if (!ep.preact) return launch_mfma_out<TM, TN, VEC, false, true>(a, m, k, b, n, kw, gw, ep, s);
    if constexpr (TM * TN < 16) return launch_mfma_out<TM, TN, VEC, true, true>(a, m, k, b, n, kw, gw, ep, s);
    else return BNN_ERR_UNSUPPORTED;
}

template <int TM, int TN>
bnn_status launch_mfma(const uint32_t *a, int64_t m, int64_t k, const uint32_t *b, int64_t n, int kw,
                       const EpiArgs &ep, hipStream_t s)
{
    GemmWalk gw;
    const int64_t nbm = ceil_div64(m, 64 * TM), nbn = ceil_div64(n, 64 * TN);
    const int64_t tiles = nbm * nbn;
    if (tiles > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
    gw.nbm = (int)nbm; gw.nbn = (int)nbn; gw.tiles = (int)tiles;
    // Streaming stores of raw sums, only of whole cache lines (6000 x 6001, K = 4096: 147 us with them, 81
    // without).  The 256 x 256 tile: where C is larger than the 256 MiB memory-side cache (12000 x 8000,
    // K = 1024: 84.5 us with, 88.5 without; 8000 x 8000, K = 512: 54 with, 48 without).  Smaller tiles: near the
    // size of that cache (5744 x 8352, K = 207 44.4 / 45.6), and in a single round, whose stores all leave at the
    // end (3000 x 3072, K = 1024 10.4 / 11.9, 1597 x 4672, K = 896 8.8 / 10.2); between them the cache takes the
    // stores faster (4096 x 4096, K = 512 16.2 / 14.9, 3020 x 8800, K = 156 26.5 / 23.6, 5657 x 6304, K = 782 35.5 / 33.3).
    const int64_t large = TM * TN < 16 ? (int64_t)3 << 24 : (int64_t)1 << 26;
    gw.stream = (n & 31) == 0 && (m * n > large || (TM * TN < 16 && tiles <= 768));
    gw.far = 64 * TM * n < (int64_t)1 << 29 ? 0 : (n < (int64_t)1 << 26 ? 1 : 2);
    if ((kw & 3) == 0) return launch_mfma_vec<TM, TN, 4>(a, m, k, b, n, kw, gw, ep, s);
    return launch_mfma_vec<TM, TN, 1>(a, m, k, b, n, kw, gw, ep, s);
}

// more than 8 rows, too few tiles for any of the three block tiles
bool fc_takes_small_kernel(int64_t m, int64_t n)
{
    return m > 8 && ceil_div64(m, 64) * ceil_div64(n, 64) < 192;
}

template <bool TAIL>
bnn_status launch_small(const uint32_t *a, int64_t m, int64_t k, const uint32_t *b, int64_t n, int kw,
                        const EpiArgs &ep, const FcTailArgs &tail, hipStream_t s)
{
    const int nbn = (int)ceil_div64(n, 32);
    const int64_t blocks = nbn * ceil_div64(m, 32);
    if (blocks > 0x7fffffffLL) return BNN_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)blocks);
    if ((kw & 3) == 0)
        hipLaunchKernelGGL((bgemm_small<4, TAIL>), grid, dim3(256), 0, s, a, b, m, n, kw, (int)k, nbn, ep, tail);
    else if ((kw & 1) == 0)
        hipLaunchKernelGGL((bgemm_small<2, TAIL>), grid, dim3(256), 0, s, a, b, m, n, kw, (int)k, nbn, ep, tail);
    else
        hipLaunchKernelGGL((bgemm_small<1, TAIL>), grid, dim3(256), 0, s, a, b, m, n, kw, (int)k, nbn, ep, tail);
    return hip_result(hipGetLastError());
}

// m <= 8 rows; the kernel is instantiated for 1, 2, 4 and 8 rows (a batch-1 launch is bound by its
// own instruction count, and the 8-row code is four times as long).
template <bool TAIL>
bnn_status launch_gemv(const uint32_t *a, int64_t m, int64_t k, const uint32_t *b, int64_t n, int kw,
                       const EpiArgs &ep, const FcTailArgs &tail, hipStream_t s)
{
    const dim3 grid((unsigned)ceil_div64(n, 32));
    const bool v4 = (kw & 3) == 0;
#define BNN_GEMV(MT)                                                                                          \
    do {                                                                                                      \
        if (v4)                                                                                               \
            hipLaunchKernelGGL((bgemv_rows<MT, 4, TAIL>), grid, dim3(512), 0, s, a, b, (int)m, n, kw, (int)k, ep, tail); \
        else                                                                                                  \
            hipLaunchKernelGGL((bgemv_rows<MT, 1, TAIL>), grid, dim3(512), 0, s, a, b, (int)m, n, kw, (int)k, ep, tail); \
    } while (0)
    if (m == 1) BNN_GEMV(1);
    else if (m == 2) BNN_GEMV(2);
    else if (m <= 4) BNN_GEMV(4);
    else BNN_GEMV(8);
#undef BNN_GEMV
    return hip_result(hipGetLastError());
}

}  // namespace

// Microseconds per 512 bits of K that the busiest compute unit spends on m x n outputs in square tiles
// of `tile`: each XCD takes an eighth of the tiles and has 32 compute units.  One 256 x 256 tile at a
// time takes 2.06, two 128 x 128 tiles side by side 1.23, one alone 0.68 (fitted to 290 products).
static double fc_tile_time(int64_t m, int64_t n, int tile)
{
    const int64_t tiles = ceil_div64(ceil_div64(m, tile) * ceil_div64(n, tile), 8);
    if (tile == 256) return 2.06 * (double)ceil_div64(tiles, 32);
    const int64_t full = tiles / 64, rest = tiles - full * 64;
    return 1.23 * (double)full + (rest == 0 ? 0.0 : (rest <= 32 ? 0.68 : 1.23));
}

int fc_binary_kernel_choice(int64_t m, int64_t k, int64_t n, bool raw, bool packed)
{
    if (m <= 8) return FC_GEMV;
    const bool both = raw && packed;                // diagnostic calls: the 256 x 256 tile would spill
    // Raw sums of millions of columns: there are tiles enough of any size, and the padding of the rows decides
    // (us, 256 x 256 / as chosen, n = 2^21: m = 9, K = 4096 847 / 374; m = 100, K = 64 390 / 180; m = 300, K = 4096
    // 1752 / 1484; at m = 512, K = 4096 the 256 x 256 tile takes 1900, the 128 x 128 one 2050).
    if (raw && n >= (int64_t)1 << 21) {
        if (m <= 64) return FC_TILE_64;
        return both || ceil_div64(m, 128) * 128 * 6 < ceil_div64(m, 256) * 256 * 5 ? FC_TILE_128 : FC_TILE_256;
    }
    // A tile has to fill most of the 256 compute units.
    const int64_t want = 192;
    if (!both && ceil_div64(m, 256) * ceil_div64(n, 256) >= want) {
        // The 256 x 256 tile multiplies fastest; the 128 x 128 tile leaves less of the last round idle, and its
        // two blocks per compute unit overlap one's stores with the other's multiplies.  us, 256 x 256 /
        // 128 x 128.  Raw sums of a short K are mostly stores: 6000 x 6000, K = 640 41.1 / 30.6, 6607 x 5280, K =
        // 1792 55.9 / 43.2, 8192 x 8192, K = 2048 87.4 / 74.2; where they are larger than the 256 MiB memory-side
        // cache the larger tile: 9000 x 9000, K = 256 97.6 / 106.5, 12000 x 8000, K = 1024 84.7 / 94.1.  Otherwise
        // the rounds decide: 7200 x 7200, K = 900 58.7 / 49.3, 8000 x 8000, K = 1024 60.0 / 61.7; with a tenth in
        // favour of the smaller tile where stores are few: 1919 x 8521, K = 6272 with step 64.8 / 42.4, 9034 x 4320,
        // K = 640 24.7 / 22.8, 4096 x 4096, K = 4096 23.9 / 26.3.
        const bool brief = raw && k <= 1024;
        if (raw && k <= 2048 && m * n <= (brief ? (int64_t)3 << 24 : (int64_t)1 << 26)) return FC_TILE_128;
        if (brief && m * n > (int64_t)1 << 26) return FC_TILE_256;
        if ((brief ? 1.0 : 1.1) * fc_tile_time(m, n, 256) <= fc_tile_time(m, n, 128)) return FC_TILE_256;
        return FC_TILE_128;
    }
    if (ceil_div64(m, 128) * ceil_div64(n, 128) >= want) return FC_TILE_128;
    // fewer than that many 64 x 64 tiles: 32 x 32 tiles with K split over the block's waves
    return fc_takes_small_kernel(m, n) ? FC_SMALL : FC_TILE_64;
}

bnn_status launch_fc_binary(const uint32_t *a, int64_t m, int64_t k, const uint32_t *b, int64_t n,
                            const EpiArgs &ep, hipStream_t s)
{
    if (m == 0) return BNN_OK;
    const int kw = (int)((k + 31) / 32);
    const FcTailArgs none = {nullptr, nullptr, 0};
    switch (fc_binary_kernel_choice(m, k, n, ep.preact != nullptr, ep.packed != nullptr)) {
    case FC_GEMV: return launch_gemv<false>(a, m, k, b, n, kw, ep, none, s);
    case FC_SMALL: return launch_small<false>(a, m, k, b, n, kw, ep, none, s);
    case FC_TILE_64: return launch_mfma<1, 1>(a, m, k, b, n, kw, ep, s);
    case FC_TILE_128: return launch_mfma<2, 2>(a, m, k, b, n, kw, ep, s);
    case FC_TILE_256: return launch_mfma<4, 4>(a, m, k, b, n, kw, ep, s);
    }
    return BNN_ERR_UNSUPPORTED;
}

bool fc_binary_tail_qualifies(int64_t m, int64_t n, int64_t n_out)
{
    if (m < 1 || n_out < 1) return false;
    // Every logit receives one atomic per 32 outputs of this layer, and additions to one address
    // queue up behind each other: beyond these widths (measured: hidden layers of 512 .. 32768
    // outputs, with and without the tail) a launch of its own for the last layer is faster.
    if (m <= 8) return m * n_out <= 512 && n <= 8192;       // bgemv_rows: one thread per (row, class)
    return fc_takes_small_kernel(m, n) && n_out <= 16 &&    // bgemm_small: two classes per thread
           n <= 1024 && m * n_out <= FC_TAIL_MAX_LOGITS;
}

bnn_status launch_fc_binary_tail(const uint32_t *a, int64_t m, int64_t k, const uint32_t *b, int64_t n,
                                 const EpiArgs &ep, const FcTailArgs &tail, hipStream_t s)
{
    if (!fc_binary_tail_qualifies(m, n, tail.n_out) || !ep.packed || !tail.w || !tail.logits)
        return BNN_ERR_UNSUPPORTED;
    const int kw = (int)((k + 31) / 32);
    if (m > 8) return launch_small<true>(a, m, k, b, n, kw, ep, tail, s);
    return launch_gemv<true>(a, m, k, b, n, kw, ep, tail, s);
}

}  // namespace bnn
