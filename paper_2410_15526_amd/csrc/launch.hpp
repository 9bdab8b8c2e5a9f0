// launch.hpp -- interface between the C ABI layer (abi.cpp) and the kernel
// launchers (*.hip).  Launchers assume validated arguments.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <tuple>

namespace sdp4 {

constexpr int kMaxPeers = 16;

// Pointer tables passed by value in the kernel arguments.
struct PeerTable {
    const void *codes[kMaxPeers];
    const float *scales[kMaxPeers];
};
struct F32Table {
    const float *p[kMaxPeers];
};

// Records `err` as the calling thread's last HIP error and returns SDP4_EHIP.
int set_hip_error(hipError_t err);

// Grids.  A launch has one block per work block: the hardware dispatches
// blocks in index order, so the chip's accesses sweep memory from front to
// back, which HBM serves faster than the scattered fronts of a persistent
// grid.  `cap` bounds the blocks resident on a compute unit at once: k >= 1
// reserves enough LDS per block that at most k fit, kUncapped leaves residency
// to the kernel's occupancy.  kPersistent: as many blocks as compute units
// (the kernel loops over its work blocks).
constexpr int kUncapped = 0;
constexpr int kPersistent = -1;

// Launches of up to this many blocks per compute unit take no cap: they are
// over in a round or two, and have no steady state for a cap to pace.  (us
// with the cap / without: 2^22 elements, 4 to 8 blocks per CU, encode 6.4 / 5.8,
// decode of float32 weights at 2^21 4.6 / 4.1, 2^23 elements, encode 10.2 / 9.8,
// K1 4-bit 8.1 / 7.8; from 12 blocks on the caps are as fast or faster.)
constexpr int kPacedBlocks = 10;

// Blocks along x; the rest go along y, since the work items of one dimension
// must stay below 2^32.  Block (x, y) is work block y * kGridX + x.
constexpr int64_t kGridXLog2 = 22, kGridX = int64_t(1) << kGridXLog2;

struct LaunchShape {
    unsigned x, y;
    size_t dyn_lds; // LDS bytes reserved per block beyond the kernel's own
};
LaunchShape shape_for(const void *kernel, int64_t nwork_blocks, int cap, hipError_t &err);

// Launch `kernel` with blocks of WAVES wavefronts.
template <int WAVES, typename... Params, typename... Args>
int launch(void (*kernel)(Params...), int64_t nwork_blocks, int cap, hipStream_t stream, Args... args)
{
    hipError_t err;
    const LaunchShape sh = shape_for(reinterpret_cast<const void *>(kernel), nwork_blocks, cap, err);
    if (err != hipSuccess)
        return set_hip_error(err);
    std::tuple<Params...> values(args...);
    void *argv[sizeof...(Params)];
    std::apply([&](auto &...v) {
        int i = 0;
        ((argv[i++] = static_cast<void *>(&v)), ...);
    }, values);
    err = hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3(sh.x, sh.y), dim3(64 * WAVES), argv,
                          sh.dyn_lds, stream);
    if (err != hipSuccess)
        return set_hip_error(err);
    return 0;
}

int launch_qwd_encode(const float *w_new, const void *w_prev, bool bf16, bool sym, int64_t n, int group,
                      uint8_t *codes, float *scale, float *minv, hipStream_t s);
int launch_qwd_decode(const uint8_t *codes, const float *scale, const float *minv, int64_t n,
                      int group, void *w_prev, bool bf16, bool sym, hipStream_t s);
int launch_grad_quant(const float *x, int64_t n, int bits, int nblk, int group, float cn,
                      uint8_t *codes, float *scale, hipStream_t s);
int launch_dequant_reduce(const PeerTable &peers, int P, int64_t n, int bits_in, int group,
                          int bits_out, int nblk, float cn, float out_scale, uint8_t *out_codes,
                          float *out_scales, float *out_f32, hipStream_t s);
int launch_dequant_reduce_f32_in8(const PeerTable &peers, int P, int64_t n, int group, int nblk, float cn,
                                  float out_scale, float *out_f32, hipStream_t s);
int launch_dequant_reduce_f32_in4(const PeerTable &peers, int P, int64_t n, int group, int nblk, float cn,
                                  float out_scale, float *out_f32, hipStream_t s);
int launch_grad_quant_sr(const float *x, int64_t n, int bits, int nblk, int group, float cn, uint64_t seed,
                         uint64_t offset, uint8_t *codes, float *scale, hipStream_t s);
int launch_dequant_reduce_sr(const PeerTable &peers, int P, int64_t n, int bits_in, int group, int bits_out,
                             uint64_t seed, uint64_t offset, uint8_t *out_codes, float *out_scales,
                             float *out_f32, hipStream_t s);
int launch_hadamard(const float *x, float *y, int64_t n, int nblk, float cn, hipStream_t s);
int launch_reduce_f32(const F32Table &xs, int P, int64_t n, float *y, hipStream_t s);
int launch_copy_f32(const float *x, float *y, int64_t n, hipStream_t s);
int launch_read_f32(const float *x, int64_t n, uint32_t *sink, hipStream_t s);
int launch_fill_f32(float *y, int64_t n, float value, hipStream_t s);

} // namespace sdp4
