// Test hook, built into tests/hooks/libbnn_test_hooks.so only: where the streamed weight transfers
// of a binary convolution read, worked out on the host with the functions that the kernel uses.
#include <vector>

#include "bconv_kernel.h"

namespace {

// Bytes past the end of the weight tensor that the transfers reach (<= 0: none), counting a transfer as
// dropped only where its vector offset alone lies past the end; *missed: words of the tensor that no
// transfer delivers.
template <int WPH>
int64_t past_end(int c_in, int c_out, int64_t *missed)
{
    using Lane = bnn::WeightLane<WPH>;
    const int cw = (c_in + 31) / 32;
    const int64_t bytes = (int64_t)c_out * 9 * cw * 4;
    const bool exact = cw == 2 * WPH && c_out % 128 == 0;
    int64_t past = -bytes;
    std::vector<bool> seen((size_t)(bytes / 4));
    for (int o_blk = 0; o_blk < c_out; o_blk += 128)
        for (int wave = 0; wave < 4; ++wave)
            for (int lane = 0; lane < 64; ++lane) {
                const Lane w(o_blk, wave, lane, cw);
                for (int chunk = 0; chunk < 9 * WPH / Lane::SPC; ++chunk)
                    for (int k = 0; k < 8; ++k) {
                        const int64_t v = exact ? w.voff_exact() : w.voff(chunk, k, cw);
                        const int64_t s = (int64_t)Lane::chunk_offset(chunk, cw) + (exact ? k * (int64_t)Lane::row_step(cw) : 0);
                        if (v >= bytes) continue;
                        if (v + s + 4 - bytes > past) past = v + s + 4 - bytes;
                        if (v + s + 4 <= bytes) seen[(size_t)((v + s) / 4)] = true;
                    }
            }
    *missed = 0;
    for (const bool b : seen) *missed += !b;
    return past;
}

}  // namespace

extern "C" int64_t bnn_test_conv_weight_reads(int c_in, int c_out, int64_t *missed)
{
    const int cw = (c_in + 31) / 32;
    if (cw > 8 && cw <= 12) return past_end<6>(c_in, c_out, missed);
    if (cw > 8 && cw <= 16) return past_end<8>(c_in, c_out, missed);
    if (cw > 16 && cw <= 32) return past_end<16>(c_in, c_out, missed);
    return -1;
}
