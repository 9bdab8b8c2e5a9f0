// k_qwd.hip -- launchers of the qWD encode and decode kernels (asymmetric
// and symmetric codecs).
#include "kernels.hpp"

namespace sdp4 {

namespace {

template <bool BF16, int WPB, bool WIDE>
int qwd_encode(const float *w_new, const void *w_prev, bool sym, int64_t n, int gs, uint8_t *codes, float *scale,
               float *minv, int cap, hipStream_t s)
{
    constexpr int E = 16;
    auto k = sym ? k_qwd_encode<BF16, true, E, WPB, WIDE> : k_qwd_encode<BF16, false, E, WPB, WIDE>;
    return launch_tiles<E, WPB>(k, n, cap, s, w_new, w_prev, n, gs, codes, scale, minv);
}

// 2-wave blocks, <= 8 per CU, 16 elements per lane for bfloat16 weights and 8 for float32: 2 KiB of weights
// read and written per wave (2^30 elements, <= 6 / 8 / 10 per CU: bfloat16 826 / 751 / 759 us, float32 <= 6 / 7 /
// 8 / 10 1526 / 1440 / 1408 / 1419).  Uncapped up to 2^23 elements (uncapped / <= 8, new inputs
// each pass: bfloat16, 5.8M 6.9 / 7.0, 7.3M 8.2 / 8.4, 2^24 14.7 / 14.8; float32, 2.9M 6.25 / 6.25, 7.3M 12.6 / 12.8,
// 2^25 46.7 / 46.9).
template <bool BF16>
int qwd_decode(const uint8_t *codes, const float *scale, const float *minv, int64_t n, int gs, void *w_prev, bool sym,
               hipStream_t s)
{
    constexpr int E = BF16 ? 16 : 8, WPB = 2;
    auto k = sym ? k_qwd_decode<BF16, true, E, WPB> : k_qwd_decode<BF16, false, E, WPB>;
    return launch_tiles<E, WPB>(k, n, n <= int64_t(1) << 23 ? kUncapped : 8, s, codes, scale, minv, n, gs, w_prev);
}

} // namespace

int launch_qwd_encode(const float *w_new, const void *w_prev, bool bf16, bool sym, int64_t n, int group,
                      uint8_t *codes, float *scale, float *minv, hipStream_t s)
{
    // 16 elements per lane, 12 waves per CU: 4-wave blocks <= 3 (2^27 elements, <= 3 / 4 / 5 / 6 per CU: bfloat16
    // weights 139.7 / 143 / 141.4 / 142.2 us, float32 179.6 / 182.4 / 184.2 / 186.0), or, for large launches with
    // bfloat16 weights, 2-wave blocks <= 6 (2^30 elements 1114 against 1145, 201M 208.7 against 210.1; 50M 53.2
    // against 53.0; float32 weights at 2^30 1465 against 1450).
    const int gs = log2_of(group);
    if (group > kWave * 16) { // beyond a wave tile; bfloat16 weights <= 4 (groups of 4096 at 1.6e9 1641, <= 3 1664),
        // or large launches whose groups two waves hold as below (2048 at 1.6e9 1699, 4-wave <= 4 1709, <= 3 1718)
        if (bf16 && group == 2048 && n >= (int64_t(1) << 28))
            return qwd_encode<true, 2, true>(w_new, w_prev, sym, n, gs, codes, scale, minv, 6, s);
        return bf16 ? qwd_encode<true, 4, true>(w_new, w_prev, sym, n, gs, codes, scale, minv, 4, s)
                    : qwd_encode<false, 4, true>(w_new, w_prev, sym, n, gs, codes, scale, minv, 3, s);
    }
    if (bf16 && n >= (int64_t(1) << 27))
        return qwd_encode<true, 2, false>(w_new, w_prev, sym, n, gs, codes, scale, minv, 6, s);
    return bf16 ? qwd_encode<true, 4, false>(w_new, w_prev, sym, n, gs, codes, scale, minv, 3, s)
                : qwd_encode<false, 4, false>(w_new, w_prev, sym, n, gs, codes, scale, minv, 3, s);
}

int launch_qwd_decode(const uint8_t *codes, const float *scale, const float *minv, int64_t n,
                      int group, void *w_prev, bool bf16, bool sym, hipStream_t s)
{
    const int gs = log2_of(group);
    return bf16 ? qwd_decode<true>(codes, scale, minv, n, gs, w_prev, sym, s)
                : qwd_decode<false>(codes, scale, minv, n, gs, w_prev, sym, s);
}

} // namespace sdp4
