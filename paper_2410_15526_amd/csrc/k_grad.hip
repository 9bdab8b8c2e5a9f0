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
        // Times in us, block 256 unless named.
        if constexpr (NB <= 256) {
            // 8 elements per lane: two stages fewer inside a lane are the DPP stages' gain, and 2 KiB read per
            // wave streams best.  8-wave blocks <= 4 per CU, or below 2^25 elements (groups that fit a wave)
            // 4-wave blocks <= 8, which spread a short launch better (8-bit, 2^21 / 2^23 / 2^24 / 2^25 / 2^27
            // elements, 8-wave 3.9 / 8.9 / 15.4 / 27.6 / 105.2, 4-wave 3.55 / 8.35 / 14.8 / 27.9 / 105.7).  16
            // per lane in 4-wave blocks, 8-bit <= 5 at 2^27 107.5; 4-bit <= 6 / 5 / 4 at 201326592 without a
            // transform 146.6 / 142.9 / 139.8, now 139.1, and with block 128 146.0 / 144.3 / 147.0, now 141.9.
            if (bits == 4)
                return few<4>(x, n, gs, cn, codes, scale, s);
            if constexpr (NB > 0)
                return few<8>(x, n, gs, cn, codes, scale, s);
            // 8-bit codes without a transform: 16 per lane, <= 4 per CU (2^27 elements <= 4 / 5 / 6 105.7 /
            // 109.5 / 110.7, 8 per lane 106.2 and 3 to 5 % slower below 2^23).
            return quantize<8, 16, 0, 4>(x, n, gs, cn, codes, scale, 4, s);
        } else {
            // Wider transforms cross rows of 16 lanes, less often the more elements a lane holds (8-bit, block
            // 512 / 1024 at 2^27: 106.9 / 107.6 with 16 per lane, 107.6 / 112 with 8).
            return bits == 4 ? quantize<4, 16, NB, 4>(x, n, gs, cn, codes, scale, 6, s)
                             : quantize<8, 16, NB, 4>(x, n, gs, cn, codes, scale, 5, s);
        }
    }

private:
    template <int BITS>
    static int few(const float *x, int64_t n, int gs, float cn, uint8_t *codes, float *scale, hipStream_t s)
    {
        constexpr int64_t M = int64_t(1) << 20;
        // Launches about what the L2s hold: 16 per lane in 4-wave blocks, uncapped (5 M elements, against 8 per
        // lane in 4-wave blocks 5.1 / 5.55 for 4 bits without a transform, 5.75 / 5.95 for 8 bits, and in 8-wave
        // blocks, for groups of 1024 and more, 5.0 / 5.6 and 5.5 / 6.05; 4 M 4.5 / 4.4, 9 M 8.1 / 8.1 and 9.2 / 9.1,
        // groups of 1024 8.75 / 9.6).
        if (n > 4 * M && n <= 9 * M)
            return quantize<BITS, 16, NB, 4>(x, n, gs, cn, codes, scale, kUncapped, s);
        if constexpr (BITS == 4) { // beyond, 4-bit codes in groups of 1024 and more, <= 6 (2048, 16 / 20 M 12.9 / 15.8
            // against 13.95 / 16.6 in 8-wave blocks; 32 M 24.4 and 24.7 with 64 points, 64 M 47.9 and 47.4 without)
            if (n > 4 * M && n < 32 * M && gs > 9)
                return quantize<4, 16, NB, 4>(x, n, gs, cn, codes, scale, 6, s);
        }
        if (n < 32 * M && gs <= 9)
            return quantize<BITS, 8, NB, 4>(x, n, gs, cn, codes, scale, 8, s);
        if constexpr (BITS == 4 && NB == 256) // 4-bit codes, 2^27 / 2^29 elements: 98.3 / 390, with 8 per lane 99.3 / 396
            return quantize<4, 16, NB, 4>(x, n, gs, cn, codes, scale, 6, s);
        else
            return quantize<BITS, 8, NB, 8>(x, n, gs, cn, codes, scale, 4, s);
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
