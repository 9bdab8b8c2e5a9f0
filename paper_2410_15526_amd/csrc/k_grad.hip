// k_grad.hip -- launchers of the Hadamard + quantization kernel (K1) and of
// the standalone Hadamard transform.
#include "kernels.hpp"

namespace sdp4 {

namespace {

template <int BITS, int E, int NB, int WPB>
int quantize(const float *x, int64_t n, int gs, float cn, uint8_t *codes, float *scale, int cap, hipStream_t s)
{
    if constexpr (kWave * E * WPB >= 4096) {
        if ((1 << gs) > kWave * E) // a group beyond a wave tile
            return launch_tiles<E, WPB>(k_grad_quant<BITS, E, NB, WPB, false, true>, n, cap, s, x, n, gs, cn, codes,
                                        scale, uint64_t(0), uint64_t(0));
    }
    return launch_tiles<E, WPB>(k_grad_quant<BITS, E, NB, WPB, false, false>, n, cap, s, x, n, gs, cn, codes, scale,
                                uint64_t(0), uint64_t(0));
}

template <int NB>
struct GradQuant {
    static int run(const float *x, int64_t n, int bits, int gs, float cn, uint8_t *codes, float *scale, hipStream_t s)
    {
        // (Times in us.)  4-bit codes: 16 elements per lane in 4-wave blocks, <= 6 per CU (32 per lane in 8-wave blocks <= 3:
        // 2^20 / 2^23 / 2^25 / 2^27 elements 4.4 / 9.0 / 26.8 / 98.0, now 3.3 / 7.8 / 25.6 / 97.7).
        if (bits == 4)
            return quantize<4, 16, NB, 4>(x, n, gs, cn, codes, scale, 6, s);
        // 8-bit codes without a transform: <= 4 per CU (<= 5 / 6: 2^27 elements 109.5 / 110.7, now 105.7).
        if constexpr (NB == 0)
            return quantize<8, 16, NB, 4>(x, n, gs, cn, codes, scale, 4, s);
        // Transforms up to 256 points: 8 elements per lane, whose two stages fewer inside a lane are the DPP
        // stages' gain; 8-wave blocks <= 4 per CU, or below 2^25 elements (groups that fit a wave) 4-wave
        // blocks <= 8, which spread a short launch better (2^21 / 2^23 / 2^24 / 2^25 / 2^27 elements, block
        // 256, 8-wave 3.9 / 8.9 / 15.4 / 27.6 / 105.2, 4-wave 3.55 / 8.35 / 14.8 / 27.9 / 105.7; 16 per lane
        // in 4-wave blocks <= 5 at 2^27 107.5).
        else if constexpr (NB <= 256)
            return n < (int64_t(1) << 25) && gs <= 9 ? quantize<8, 8, NB, 4>(x, n, gs, cn, codes, scale, 8, s)
                                                     : quantize<8, 8, NB, 8>(x, n, gs, cn, codes, scale, 4, s);
        // Wider ones cross rows of 16 lanes, the fewer the more elements a lane holds (block 512 / 1024 at
        // 2^27: 106.9 / 107.6 with 16 per lane, 107.6 / 112 with 8).
        else
            return quantize<8, 16, NB, 4>(x, n, gs, cn, codes, scale, 5, s);
    }
};

template <int NB>
struct Hadamard {
    static int run(const float *x, float *y, int64_t n, float cn, hipStream_t s)
    {
        if constexpr (NB < 2)
            return 1;
        else
            return launch_tiles<16, 4>(k_hadamard<16, NB, 4>, n, 4, s, x, y, n, cn);
    }
};

} // namespace

int launch_grad_quant(const float *x, int64_t n, int bits, int nblk, int group, float cn,
                      uint8_t *codes, float *scale, hipStream_t s)
{
    return with_block<GradQuant>(nblk, x, n, bits, log2_of(group), cn, codes, scale, s);
}

int launch_hadamard(const float *x, float *y, int64_t n, int nblk, float cn, hipStream_t s)
{
    return with_block<Hadamard>(nblk, x, y, n, cn, s);
}

} // namespace sdp4
