// k_sr.hip -- launchers of the stochastically rounded gradient quantizers:
// Hadamard + quantization (K1) and dequantize-reduce + re-quantization (K2).
#include "kernels.hpp"

namespace sdp4 {

namespace {

template <int BITS, int E, int NB, int WPB>
int quantize_sr(const float *x, int64_t n, int gs, float cn, uint64_t seed, uint64_t offset, uint8_t *codes,
                float *scale, int cap, hipStream_t s)
{
    auto k = (1 << gs) > kWave * E ? k_grad_quant<BITS, E, NB, WPB, true, true>
                                   : k_grad_quant<BITS, E, NB, WPB, true, false>;
    return launch_tiles<E, WPB>(k, n, cap, s, x, n, gs, cn, codes, scale, seed, offset);
}

// 16 elements per lane in 4-wave blocks, <= 6 per CU, where the transform adds to the generator's work; with at
// most 32 points and 8-bit codes HBM bounds it, and 8 per lane in 8-wave blocks are faster (2^27 elements, block
// 0 / 32 / 128 / 256: 104.1 / 105.0 / 110.5 / 113.5 us, 16 per lane 110.2 / 109.8 / 109.1 / 106.2).
template <int NB>
struct GradQuantSR {
    static int run(const float *x, int64_t n, int bits, int gs, float cn, uint64_t seed, uint64_t offset,
                   uint8_t *codes, float *scale, hipStream_t s)
    {
        if (bits == 4)
            return quantize_sr<4, 16, NB, 4>(x, n, gs, cn, seed, offset, codes, scale, 6, s);
        if constexpr (NB <= 32)
            return quantize_sr<8, 8, NB, 8>(x, n, gs, cn, seed, offset, codes, scale, kUncapped, s);
        else
            return quantize_sr<8, 16, NB, 4>(x, n, gs, cn, seed, offset, codes, scale, 6, s);
    }
};

} // namespace

int launch_grad_quant_sr(const float *x, int64_t n, int bits, int nblk, int group, float cn, uint64_t seed,
                         uint64_t offset, uint8_t *codes, float *scale, hipStream_t s)
{
    return with_block<GradQuantSR>(nblk, x, n, bits, log2_of(group), cn, seed, offset, codes, scale, s);
}

int launch_dequant_reduce_sr(const PeerTable &peers, int P, int64_t n, int bits_in, int group, int bits_out,
                             uint64_t seed, uint64_t offset, uint8_t *out_codes, float *out_scales,
                             float *out_f32, hipStream_t s)
{
    const int gs = log2_of(group);
    if (bits_in == 8)
        return bits_out == 4
                   ? requant_for<8, 4, true>(peers, P, n, gs, out_codes, out_scales, out_f32, s, seed, offset)
                   : requant_for<8, 8, true>(peers, P, n, gs, out_codes, out_scales, out_f32, s, seed, offset);
    return bits_out == 4
               ? requant_for<4, 4, true>(peers, P, n, gs, out_codes, out_scales, out_f32, s, seed, offset)
               : requant_for<4, 8, true>(peers, P, n, gs, out_codes, out_scales, out_f32, s, seed, offset);
}

} // namespace sdp4
