// kernels.hpp -- gfx950 kernel templates of the SDP4Bit compression hot
// path; the .hip files instantiate and launch them.
//
// One wave tile of 64*E consecutive elements per wavefront (see device.hpp
// for the lane layout), one launch block per WPB tiles, no loop: the
// hardware dispatches blocks in index order, so the chip's accesses sweep
// memory front to back, which HBM serves faster than the scattered fronts
// of a persistent grid.  All blocks but the last are whole, which is decided
// once per block on scalars; a whole block's code has no bounds checks and
// addresses memory as a scalar base plus a 32-bit lane offset, so its first
// load goes out after a few instructions and the LDS addresses and constants
// are computed while it is in flight.  (As loops over tiles, the kernels
// spent 100 to 160 vector instructions per wave before the first load on
// values hoisted out of a loop that ran once.  Against those: 2^20 elements,
// encode 3.5 -> 3.1 us, K1 3.2 -> 2.9, K2 with 8 peers 4.1 -> 3.1; above
// 2^27 elements, where HBM bounds them, within 2 %.)
//
// A quantization group that fits a wave tile is reduced with cross-lane
// exchanges; a larger one (WIDE) spans 2 to 8 whole waves of one block, which
// exchange one value each through LDS and a barrier.  (With the group in one
// wave, 64 elements per lane, groups of 4096 ran at 36 to 80 % of the other
// groups' rate: too few and too heavy waves.)
//
// Block shapes: waves per block, and a cap on the blocks resident on a
// compute unit at once (launch.hpp).  How many bytes a CU keeps in flight
// moves the mixed read/write bandwidth of HBM by several per cent; each cap
// says what it was measured against.
#pragma once

#include "device.hpp"
#include "launch.hpp"

#include <type_traits>

namespace sdp4 {

// ---------------------------------------------------------------------------
// One tile per wave
// ---------------------------------------------------------------------------
// Where a wave's tile lies: block base (uniform) plus wave and lane.
template <int E, int WPB>
struct Place {
    static constexpr int W = kWave * E; // elements per wave tile
    static constexpr int BT = W * WPB;  // elements per block
    int64_t base;                       // first element of the block
    int64_t rest;                       // elements from there to the end (may be none)
    uint32_t wave, lane;
    SDP4_DEV explicit Place(int64_t n)
        : base(((int64_t)blockIdx.y << kGridXLog2 | blockIdx.x) * BT), rest(n - base), wave(threadIdx.x / kWave), lane(threadIdx.x % kWave)
    {
    }
    SDP4_DEV bool whole() const { return rest >= BT; }
    // elements of this wave's tile, 0 past the end
    SDP4_DEV int valid() const
    {
        const int64_t r = rest - (int)(wave * W);
        return (int)(r < 0 ? 0 : r < W ? r : W);
    }
    // Offset of the block in its group: groups are at most 4096 elements, so
    // smaller blocks may start inside one.
    SDP4_DEV uint32_t in_group(int gs) const { return BT >= 4096 ? 0u : (uint32_t)base & ((1u << gs) - 1); }
};

// Two copies of the body, for whole blocks and for the last, partial one.
template <class F>
SDP4_DEV void whole_or_partial(bool whole, F body)
{
    if (whole)
        body(std::true_type{});
    else
        body(std::false_type{});
}

// Coalesced 16-byte chunks of a wave tile (R per lane) that starts at chunk
// wave*64*R of `block`; chunks at or beyond `valid` (of the tile) are zero.
template <bool WHOLE, int R>
SDP4_DEV void load_chunks(const void *block, uint32_t wave, uint32_t lane, int valid, u32x4 (&t)[R])
{
    const char *p = static_cast<const char *>(block) + (wave * (kWave * R) + lane) * 16u;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        if (WHOLE || (int)lane + kWave * i < valid)
            t[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p + i * (kWave * 16)));
        else
            t[i] = u32x4{0u, 0u, 0u, 0u};
    }
}

// The reverse, from the lane-contiguous layout (element lane el).
template <bool WHOLE, int R>
SDP4_DEV void store_chunks(void *block, uint32_t wave, uint32_t lane, int valid, u32x4 *lds, const u32x4 (&in)[R], int el)
{
#pragma unroll
    for (int k = 0; k < R; ++k)
        lds[swz<R>(R * el + k)] = in[k];
    wave_lds_sync();
    char *p = static_cast<char *>(block) + (wave * (kWave * R) + lane) * 16u;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int c = kWave * i + (int)lane;
        const u32x4 t = lds[swz<R>(c)];
        if (WHOLE || c < valid)
            __builtin_nontemporal_store(t, reinterpret_cast<u32x4 *>(p + i * (kWave * 16)));
    }
}

// WORDS consecutive 32-bit words (1, 2 or a multiple of 4, aligned to their size up to 16 bytes).
template <int WORDS>
SDP4_DEV void load_words(const char *p, uint32_t (&w)[WORDS])
{
    if constexpr (WORDS == 1) {
        w[0] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p));
    } else if constexpr (WORDS == 2) {
        const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(p));
        w[0] = v.x, w[1] = v.y;
    } else {
#pragma unroll
        for (int k = 0; k < WORDS / 4; ++k) {
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p) + k);
            w[4 * k] = v.x, w[4 * k + 1] = v.y, w[4 * k + 2] = v.z, w[4 * k + 3] = v.w;
        }
    }
}

// Header `gi` of the group headers that start at `block`.
SDP4_DEV float load_header(const float *block, uint32_t gi)
{
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(block) + gi * 4u);
}

SDP4_DEV void store_header(float *block, uint32_t gi, float v)
{
    *reinterpret_cast<float *>(reinterpret_cast<char *>(block) + gi * 4u) = v;
}

// Pack and store the codes of a tile (E * BITS / 8 bytes of lane el): up to 16 bytes
// per lane go out directly, more through LDS so that every store instruction
// writes 1 KiB contiguous.
template <int E, int BITS, bool WHOLE>
SDP4_DEV void store_codes(uint8_t *block, uint32_t wave, uint32_t lane, int valid, u32x4 *lds, const uint32_t (&q)[E],
                          int el)
{
    constexpr int WORDS = E * BITS / 32;
    uint32_t w[WORDS];
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
        if constexpr (BITS == 4)
            w[k] = pack_nibbles8(q + 8 * k);
        else
            w[k] = pack_bytes4(q[4 * k], q[4 * k + 1], q[4 * k + 2], q[4 * k + 3]);
    }
    if constexpr (WORDS > 4) {
        u32x4 pk[WORDS / 4];
#pragma unroll
        for (int k = 0; k < WORDS / 4; ++k)
            pk[k] = u32x4{w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]};
        store_chunks<WHOLE>(block, wave, lane, valid * BITS / 128, lds, pk, el);
    } else if (WHOLE || E * el < valid) {
        char *p = reinterpret_cast<char *>(block) + (wave * kWave + el) * (WORDS * 4u);
        if constexpr (WORDS == 1)
            __builtin_nontemporal_store(w[0], reinterpret_cast<uint32_t *>(p));
        else if constexpr (WORDS == 2)
            __builtin_nontemporal_store(u32x2{w[0], w[1]}, reinterpret_cast<u32x2 *>(p));
        else
            __builtin_nontemporal_store(u32x4{w[0], w[1], w[2], w[3]}, reinterpret_cast<u32x4 *>(p));
    }
}

// First wave and number of waves of the (wide) group that `wave` belongs to.
template <int E>
SDP4_DEV uint32_t group_waves(int gs) { return (1u << gs) / (kWave * E); }

// Largest magnitude of each lane's group, from each lane's own.
template <int E, bool WIDE>
SDP4_DEV void group_max(float &a, int gs, uint32_t wave, float *red)
{
    if constexpr (!WIDE) {
        max_lanes(a, (1 << gs) / E);
    } else {
        max_lanes(a, kWave);
        red[wave] = a;
        __syncthreads();
        const uint32_t gw = group_waves<E>(gs), w0 = wave & ~(gw - 1);
        for (uint32_t k = 0; k < gw; ++k)
            a = fmaxf(a, red[w0 + k]);
    }
}

// Smallest and largest value of each lane's group.
template <int E, bool WIDE>
SDP4_DEV void group_minmax(float &mn, float &mx, int gs, uint32_t wave, float *red)
{
    if constexpr (!WIDE) {
        minmax_lanes(mn, mx, (1 << gs) / E);
    } else {
        minmax_lanes(mn, mx, kWave);
        red[2 * wave] = mn;
        red[2 * wave + 1] = mx;
        __syncthreads();
        const uint32_t gw = group_waves<E>(gs), w0 = wave & ~(gw - 1);
        for (uint32_t k = 0; k < gw; ++k) {
            mn = fminf(mn, red[2 * (w0 + k)]);
            mx = fmaxf(mx, red[2 * (w0 + k) + 1]);
        }
    }
}

template <int E>
SDP4_DEV float largest(const float (&v)[E])
{
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < E; ++i)
        a = fmaxf(a, fabsf(v[i]));
    return a;
}

// Symmetric codes of E elements, rounded to nearest or (SR) stochastically
// with the uniforms of elements e0 and up.
template <int E, bool SR>
SDP4_DEV void sym_codes(const float (&v)[E], float inv, float qmax, uint64_t seed, uint64_t e0, uint32_t (&q)[E])
{
    if constexpr (SR) {
        float h[E];
        sr_uniforms<E>(seed, e0, h);
#pragma unroll
        for (int i = 0; i < E; ++i)
            q[i] = code_bits_sr(v[i], inv, h[i], (int)qmax);
    } else {
#pragma unroll
        for (int i = 0; i < E; ++i)
            q[i] = code_bits(v[i], inv);
    }
}

// Fused transform of a kernel whose lanes follow element_lane when blocks
// span several lanes (NB > E); within one lane, the plain transform; none for NB = 0.
template <int E, int NB>
SDP4_DEV void fused_fwht(float (&v)[E], float cn, int el)
{
    if constexpr (NB > E)
        fwht_lane_signed<E, NB>(v, cn, el);
    else if constexpr (NB > 1)
        fwht_lane<E, NB>(v, cn);
}

// ---------------------------------------------------------------------------
// qWD encode: d = w_new - widen(w_prev); 4-bit codes per group, asymmetric
// (codes 0..15, scale and minimum) or, with SYM, symmetric (codes -7..7,
// scale only; minv is not touched).  Bound by HBM, whose rate depends on how
// many bytes the waves keep in flight; the launcher's cap sets that.  (A form
// that read and wrote in alternating phases of the wall clock, buffering
// codes in LDS, was slower at every size: bfloat16 weights, 2^26 / 2^27 / 2^30
// elements, 75.0 / 145 / 1157 us against 70.6 / 139.8 / 1145.)
// ---------------------------------------------------------------------------
template <bool BF16, bool SYM, int E, int WPB, bool WIDE>
__global__ __launch_bounds__(kWave * WPB) void k_qwd_encode(
    const float *__restrict__ w_new, const void *__restrict__ w_prev, int64_t n, int gs,
    uint8_t *__restrict__ codes, float *__restrict__ scale, float *__restrict__ minv)
{
    using Pl = Place<E, WPB>;
    static_assert(!WIDE || Pl::BT >= 2048, "a group (2 waves: of at most 2048 elements) within one block");
    constexpr int R = E / 4;
    constexpr int RP = BF16 ? E / 8 : E / 4;
    __shared__ u32x4 lds_all[WPB][kWave * R];
    __shared__ float red[WIDE ? 2 * WPB : 1];
    const Pl at(n);
    u32x4 *lds = lds_all[at.wave];
    whole_or_partial(at.whole(), [&](auto w) {
        constexpr bool WHOLE = decltype(w)::value;
        const int valid = WHOLE ? Pl::W : at.valid();
        u32x4 ta[R], tb[RP];
        load_chunks<WHOLE>(w_new + at.base, at.wave, at.lane, valid / 4, ta);
        if constexpr (BF16)
            load_chunks<WHOLE>(static_cast<const uint16_t *>(w_prev) + at.base, at.wave, at.lane, valid / 8, tb);
        else
            load_chunks<WHOLE>(static_cast<const float *>(w_prev) + at.base, at.wave, at.lane, valid / 4, tb);
        float d[E], p[E];
        {
            u32x4 c[R];
            transpose_in<R>(ta, lds, c, at.lane);
            chunks_to_f32<E>(c, d);
        }
        {
            u32x4 c[RP];
            transpose_in<RP>(tb, lds, c, at.lane);
            if constexpr (BF16)
                bf16_chunks_to_f32<E>(c, p);
            else
                chunks_to_f32<E>(c, p);
        }
#pragma unroll
        for (int i = 0; i < E; ++i)
            d[i] = d[i] - p[i];
        uint32_t q[E];
        float s, mn = 0.0f;
        if constexpr (SYM) {
            float a = largest(d);
            group_max<E, WIDE>(a, gs, at.wave, red);
            float inv;
            sym_params(a, 7.0f, s, inv);
#pragma unroll
            for (int i = 0; i < E; ++i)
                q[i] = code_bits(d[i], inv);
        } else {
            mn = d[0];
            float mx = d[0];
#pragma unroll
            for (int i = 1; i < E; ++i) {
                mn = fminf(mn, d[i]);
                mx = fmaxf(mx, d[i]);
            }
            group_minmax<E, WIDE>(mn, mx, gs, at.wave, red);
            const float range = mx - mn;
            const float r = 15.0f / range;
            const bool degenerate = !(range > 0.0f) || !__builtin_isfinite(range) || !__builtin_isfinite(r);
            s = degenerate ? 0.0f : range / 15.0f;
            const float inv = degenerate ? 0.0f : r;
#pragma unroll
            for (int i = 0; i < E; ++i)
                q[i] = code_bits(d[i] - mn, inv);
        }
        store_codes<E, 4, WHOLE>(codes + at.base / 2, at.wave, at.lane, valid, lds, q, at.lane);
        const uint32_t off = at.wave * Pl::W + E * at.lane;
        const uint32_t rem = at.in_group(gs);
        if ((WHOLE || (int)(E * at.lane) < valid) && ((off + rem) & ((1u << gs) - 1)) == 0) {
            const uint32_t gi = (off + rem) >> gs;
            store_header(scale + (at.base >> gs), gi, s);
            if constexpr (!SYM)
                store_header(minv + (at.base >> gs), gi, mn);
        }
    });
}

// ---------------------------------------------------------------------------
// qWD decode: w_prev <- narrow(widen(w_prev) + value) with value =
// fma(code, scale, min), or with SYM value = code * scale (signed codes,
// minv not read).  Bound by HBM: as many bytes written as weights read.
// ---------------------------------------------------------------------------
template <bool BF16, bool SYM, int E, int WPB>
__global__ __launch_bounds__(kWave * WPB) void k_qwd_decode(
    const uint8_t *__restrict__ codes, const float *__restrict__ scale,
    const float *__restrict__ minv, int64_t n, int gs, void *__restrict__ w_prev)
{
    static_assert(E == 8 || E == 16, "lane slice");
    using Pl = Place<E, WPB>;
    constexpr int RP = BF16 ? E / 8 : E / 4;   // 16-byte chunks of weights per lane
    constexpr int CWD = E / 8;                 // 32-bit words of codes per lane
    __shared__ u32x4 lds_all[WPB][kWave * RP];
    const Pl at(n);
    u32x4 *lds = lds_all[at.wave];
    whole_or_partial(at.whole(), [&](auto wh) {
        constexpr bool WHOLE = decltype(wh)::value;
        const int valid = WHOLE ? Pl::W : at.valid();
        u32x4 tw[RP];
        uint32_t cw[CWD] = {};
        float s = 0.0f, mn = 0.0f;
        void *wb = BF16 ? static_cast<void *>(static_cast<uint16_t *>(w_prev) + at.base)
                        : static_cast<void *>(static_cast<float *>(w_prev) + at.base);
        constexpr int per = BF16 ? 8 : 4;
        const uint32_t rem = at.in_group(gs);
        const uint32_t gi = (at.wave * Pl::W + E * at.lane + rem) >> gs;
        load_chunks<WHOLE>(wb, at.wave, at.lane, valid / per, tw); // first: the transposition waits for them alone
        if (WHOLE || (int)(E * at.lane) < valid) {
            load_words<CWD>(reinterpret_cast<const char *>(codes + at.base / 2) + (at.wave * kWave + at.lane) * (CWD * 4u), cw);
            s = load_header(scale + (at.base >> gs), gi);
            if constexpr (!SYM)
                mn = load_header(minv + (at.base >> gs), gi);
        }
        float w[E];
        u32x4 c[RP];
        transpose_in<RP>(tw, lds, c, at.lane);
        if constexpr (BF16)
            bf16_chunks_to_f32<E>(c, w);
        else
            chunks_to_f32<E>(c, w);
#pragma unroll
        for (int k = 0; k < CWD; ++k) { // word k: the nibbles of elements 8k .. 8k+7, even ones low
            const uint32_t word = cw[k];
            if constexpr (SYM) {
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const float code = (float)((int32_t)(word << (28 - 4 * m)) >> 28);
                    const float value = code * s;
                    w[8 * k + m] = w[8 * k + m] + value;
                }
            } else {
                // byte j of lo / hi: the code of element 8k + 2j / 8k + 2j + 1
                const uint32_t lo = word & 0x0F0F0F0Fu, hi = (word >> 4) & 0x0F0F0F0Fu;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float c0 = (float)((lo >> (8 * j)) & 0xFFu), c1 = (float)((hi >> (8 * j)) & 0xFFu);
                    w[8 * k + 2 * j] = w[8 * k + 2 * j] + __builtin_fmaf(c0, s, mn);
                    w[8 * k + 2 * j + 1] = w[8 * k + 2 * j + 1] + __builtin_fmaf(c1, s, mn);
                }
            }
        }
        if constexpr (BF16)
            f32_to_bf16_chunks<E>(w, c);
        else
            f32_to_chunks<E>(w, c);
        store_chunks<WHOLE>(wb, at.wave, at.lane, valid / per, lds, c, at.lane);
    });
}

// ---------------------------------------------------------------------------
// K1: blockwise Hadamard (block NB, 0 = none) + symmetric BITS-bit group
// quantization.  Bound by HBM at the launchers' shapes (5.9-6.4 TB/s of its
// bytes from 2^27 elements on); with SR by the generator's instructions.
// ---------------------------------------------------------------------------
template <int BITS, int E, int NB, int WPB, bool SR, bool WIDE>
__global__ __launch_bounds__(kWave * WPB) void k_grad_quant(
    const float *__restrict__ x, int64_t n, int gs, float cn, uint8_t *__restrict__ codes,
    float *__restrict__ scale, uint64_t seed = 0, uint64_t offset = 0)
{
    using Pl = Place<E, WPB>;
    static_assert(!WIDE || Pl::BT >= 4096, "a group within one block");
    constexpr int R = E / 4;
    constexpr float qmax = BITS == 8 ? 127.0f : 7.0f;
    __shared__ u32x4 lds_all[WPB][kWave * R];
    __shared__ float red[WIDE ? WPB : 1];
    const Pl at(n);
    u32x4 *lds = lds_all[at.wave];
    whole_or_partial(at.whole(), [&](auto w) {
        constexpr bool WHOLE = decltype(w)::value;
        const int valid = WHOLE ? Pl::W : at.valid();
        u32x4 t[R];
        load_chunks<WHOLE>(x + at.base, at.wave, at.lane, valid / 4, t);
        const int el = NB > E ? element_lane(at.lane) : at.lane; // element lane of this lane
        float v[E];
        {
            u32x4 c[R];
            transpose_in<R>(t, lds, c, el);
            chunks_to_f32<E>(c, v);
        }
        fused_fwht<E, NB>(v, cn, el);
        float a = largest(v);
        group_max<E, WIDE>(a, gs, at.wave, red);
        float s, inv;
        sym_params(a, qmax, s, inv);
        uint32_t q[E];
        const uint32_t off = at.wave * Pl::W + E * el;
        sym_codes<E, SR>(v, inv, qmax, seed, offset + (uint64_t)at.base + off, q);
        store_codes<E, BITS, WHOLE>(codes + at.base * BITS / 8, at.wave, at.lane, valid, lds, q, el);
        const uint32_t rem = at.in_group(gs);
        if ((WHOLE || E * el < valid) && ((off + rem) & ((1u << gs) - 1)) == 0)
            store_header(scale + (at.base >> gs), (off + rem) >> gs, s);
    });
}

// ---------------------------------------------------------------------------
// K2 / K3: dequantize + reduce over P <= PMAX chunks (EXACT: P == PMAX, no
// tests of P), then re-quantize (k_requant) or inverse Hadamard (block NB)
// and out_scale to float32 (k_reduce_to_f32)
// ---------------------------------------------------------------------------
// Sum over the peers, in order, of this lane's E elements.  EXACT: there are
// PMAX peers, else P <= PMAX.
template <int BITS, int E, int PMAX, bool EXACT, bool WHOLE>
SDP4_DEV void reduce_peers(const PeerTable &peers, int P, int64_t base, uint32_t off, uint32_t gi, int64_t gbase,
                           bool active, float (&acc)[E])
{
    constexpr int WORDS = E * BITS / 32;
    uint32_t c[PMAX][WORDS] = {};
    float s[PMAX] = {};
    if (WHOLE || active) {
#pragma unroll
        for (int j = 0; j < PMAX; ++j) {
            if (EXACT || j < P) {
                load_words<WORDS>(static_cast<const char *>(peers.codes[j]) + base * BITS / 8 + off * BITS / 8, c[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < PMAX; ++j)
            if (EXACT || j < P)
                s[j] = load_header(peers.scales[j] + gbase, gi);
    }
#pragma unroll
    for (int i = 0; i < E; ++i)
        acc[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < PMAX; ++j) {
        if (EXACT || j < P) {
            if constexpr (BITS == 4) {
#pragma unroll
                for (int k = 0; k < WORDS; ++k)
                    fma_codes4(c[j][k], s[j], acc + 8 * k);
            } else {
#pragma unroll
                for (int i = 0; i < E; ++i)
                    acc[i] = __builtin_fmaf(code8_f(c[j], i), s[j], acc[i]);
            }
        }
    }
}

template <int BITS_IN, int BITS_OUT, int E, int PMAX, bool EXACT, int WPB, bool SR, bool WIDE>
__global__ __launch_bounds__(kWave * WPB) void k_requant(
    PeerTable peers, int P, int64_t n, int gs, uint8_t *__restrict__ out_codes, float *__restrict__ out_scales,
    float *__restrict__ out_f32, uint64_t seed, uint64_t offset)
{
    using Pl = Place<E, WPB>;
    static_assert(Pl::BT >= 4096, "a group within one block");
    constexpr bool F32 = !EXACT; // the optional float32 output
    constexpr int R = E / 4;
    constexpr bool LDS = F32 || E * BITS_OUT > 128;
    __shared__ u32x4 lds_all[LDS ? WPB : 1][LDS ? kWave * R : 1];
    __shared__ float red[WIDE ? WPB : 1];
    const Pl at(n);
    u32x4 *lds = lds_all[LDS ? at.wave : 0];
    whole_or_partial(at.whole(), [&](auto w) {
        constexpr bool WHOLE = decltype(w)::value;
        const int valid = WHOLE ? Pl::W : at.valid();
        const int el = at.lane;
        const bool active = WHOLE || E * el < valid;
        const uint32_t off = at.wave * Pl::W + E * el;
        float acc[E];
        reduce_peers<BITS_IN, E, PMAX, EXACT, WHOLE>(peers, P, at.base, off, off >> gs, at.base >> gs, active, acc);
        if constexpr (F32) {
            if (out_f32) {
                u32x4 c[R];
                f32_to_chunks<E>(acc, c);
                store_chunks<WHOLE>(out_f32 + at.base, at.wave, at.lane, valid / 4, lds, c, el);
                wave_lds_sync();
            }
        }
        constexpr float qmax = BITS_OUT == 8 ? 127.0f : 7.0f;
        float a = largest(acc);
        group_max<E, WIDE>(a, gs, at.wave, red);
        float s, inv;
        sym_params(a, qmax, s, inv);
        uint32_t q[E];
        sym_codes<E, SR>(acc, inv, qmax, seed, offset + (uint64_t)at.base + off, q);
        store_codes<E, BITS_OUT, WHOLE>(out_codes + at.base * BITS_OUT / 8, at.wave, at.lane, valid, lds, q, el);
        if (active && (off & ((1u << gs) - 1)) == 0)
            store_header(out_scales + (at.base >> gs), off >> gs, s);
    });
}

template <int BITS_IN, int E, int NB, int PMAX, bool EXACT, int WPB>
__global__ __launch_bounds__(kWave * WPB) void k_reduce_to_f32(
    PeerTable peers, int P, int64_t n, int gs, float cn, float out_scale, float *__restrict__ out_f32)
{
    using Pl = Place<E, WPB>;
    constexpr int R = E / 4;
    __shared__ u32x4 lds_all[WPB][kWave * R];
    const Pl at(n);
    u32x4 *lds = lds_all[at.wave];
    whole_or_partial(at.whole(), [&](auto w) {
        constexpr bool WHOLE = decltype(w)::value;
        const int valid = WHOLE ? Pl::W : at.valid();
        const int el = NB > E ? element_lane(at.lane) : at.lane; // relabeled when the transform spans lanes
        const uint32_t off = at.wave * Pl::W + E * el;
        const uint32_t rem = at.in_group(gs);
        float acc[E];
        reduce_peers<BITS_IN, E, PMAX, EXACT, WHOLE>(peers, P, at.base, off, (off + rem) >> gs, at.base >> gs,
                                                     WHOLE || E * el < valid, acc);
        fused_fwht<E, NB>(acc, cn, el);
        if (out_scale != 1.0f) {
#pragma unroll
            for (int i = 0; i < E; ++i)
                acc[i] = acc[i] * out_scale;
        }
        u32x4 c[R];
        f32_to_chunks<E>(acc, c);
        store_chunks<WHOLE>(out_f32 + at.base, at.wave, at.lane, valid / 4, lds, c, el);
    });
}

// ---------------------------------------------------------------------------
// standalone Hadamard (unfused variant); in place allowed
// ---------------------------------------------------------------------------
template <int E, int NB, int WPB>
__global__ __launch_bounds__(kWave * WPB) void k_hadamard(const float *x, float *y, int64_t n, float cn)
{
    using Pl = Place<E, WPB>;
    constexpr int R = E / 4;
    __shared__ u32x4 lds_all[WPB][kWave * R];
    const Pl at(n);
    u32x4 *lds = lds_all[at.wave];
    whole_or_partial(at.whole(), [&](auto w) {
        constexpr bool WHOLE = decltype(w)::value;
        const int valid = WHOLE ? Pl::W : at.valid();
        u32x4 t[R], c[R];
        load_chunks<WHOLE>(x + at.base, at.wave, at.lane, valid / 4, t);
        transpose_in<R>(t, lds, c, at.lane);
        float v[E];
        chunks_to_f32<E>(c, v);
        fwht_lane<E, NB>(v, cn);
        f32_to_chunks<E>(v, c);
        store_chunks<WHOLE>(y + at.base, at.wave, at.lane, valid / 4, lds, c, at.lane);
        if constexpr (NB == 2 && !WHOLE) { // 16-byte chunks leave the last pair of n = 4k + 2 elements
            if (valid % 4 != 0 && at.lane == 0) {
                const int64_t i = at.base + at.wave * Pl::W + valid - 2;
                const float a = x[i], b = x[i + 1];
                y[i] = (a + b) * cn;
                y[i + 1] = (a - b) * cn;
            }
        }
    });
}

// ---------------------------------------------------------------------------
// launch helpers shared by the .hip translation units
// ---------------------------------------------------------------------------
inline int log2_of(int group) { return __builtin_ctz((unsigned)group); }

// Hadamard block sizes the kernels are compiled for: 0 (none), 2 .. 1024.
template <template <int> class F, typename... A>
int with_block(int nb, A... a)
{
    switch (nb) {
    case 0: return F<0>::run(a...);
    case 2: return F<2>::run(a...);
    case 4: return F<4>::run(a...);
    case 8: return F<8>::run(a...);
    case 16: return F<16>::run(a...);
    case 32: return F<32>::run(a...);
    case 64: return F<64>::run(a...);
    case 128: return F<128>::run(a...);
    case 256: return F<256>::run(a...);
    case 512: return F<512>::run(a...);
    case 1024: return F<1024>::run(a...);
    default: return 1;
    }
}

// Launch a kernel of one tile of 64*E elements per wave, WPB waves per block,
// at most `cap` blocks (kUncapped: as many as fit) resident on a compute unit.
template <int E, int WPB, typename... Params, typename... Args>
int launch_tiles(void (*kernel)(Params...), int64_t n, int cap, hipStream_t s, Args... args)
{
    constexpr int64_t BT = (int64_t)kWave * E * WPB;
    return launch<WPB>(kernel, (n + BT - 1) / BT, cap, s, args...);
}

// A set of peer counts: bit p for p peers.
constexpr uint32_t peer_range(int lo, int hi) { return (2u << hi) - (1u << lo); }
constexpr uint32_t kAllPeers = peer_range(1, 16);

// Calls `go` with the kernel for P peers, a count of the set PEERS: K<PMAX,
// EXACT>::get() is one with PMAX peers (EXACT) or with up to PMAX.  1 to 8 and
// 16 peers have instantiations of their own, without tests of P between the
// loads (2^27 input elements, against the guarded form on the same box: 4 to 4
// bits 18.6 -> 17.5 us with 4 peers and 18.0 -> 16.0 with 16, 8 to 4 bits of
// small chunks 3.6 -> 3.2); other counts take the guarded one of 16.
template <template <int, bool> class K, uint32_t PEERS, class Go>
int with_peers(int P, Go go)
{
    const auto exact = [&](auto count, int &rc) {
        constexpr int N = decltype(count)::value;
        if constexpr (PEERS >> N & 1) {
            if (P == N) {
                rc = go(K<N, true>::get());
                return true;
            }
        }
        return false;
    };
    int rc = 0;
    if (exact(std::integral_constant<int, 1>{}, rc) || exact(std::integral_constant<int, 2>{}, rc) ||
        exact(std::integral_constant<int, 3>{}, rc) || exact(std::integral_constant<int, 4>{}, rc) ||
        exact(std::integral_constant<int, 5>{}, rc) || exact(std::integral_constant<int, 6>{}, rc) ||
        exact(std::integral_constant<int, 7>{}, rc) || exact(std::integral_constant<int, 8>{}, rc) ||
        exact(std::integral_constant<int, 16>{}, rc))
        return rc;
    if constexpr (PEERS & peer_range(9, 15))
        return go(K<16, false>::get());
    return 1; // not reached: P is in PEERS
}

// The same with the guarded kernels only, of up to 4, 8 or 16 peers.
template <template <int, bool> class K, uint32_t PEERS, class Go>
int with_guarded_peers(int P, Go go)
{
    if constexpr (PEERS & peer_range(1, 4)) {
        if (P <= 4)
            return go(K<4, false>::get());
    }
    if constexpr (PEERS & peer_range(5, 8)) {
        if (P <= 8)
            return go(K<8, false>::get());
    }
    if constexpr (PEERS & peer_range(9, 16))
        return go(K<16, false>::get());
    return 1; // not reached: P is in PEERS
}

template <int BITS_IN, int BITS_OUT, int E, int WPB, bool SR, bool WIDE>
struct Requant {
    template <int PMAX, bool EXACT>
    struct Kernel {
        static auto get() { return k_requant<BITS_IN, BITS_OUT, E, PMAX, EXACT, WPB, SR, WIDE>; }
    };
};

// Shapes of the re-quantizing dequantize-reduce (us; M = 2^20 elements of a chunk).
//
// 8-bit messages: 16 elements per lane, one 16-byte chunk per peer; a wave
// keeps P KiB in flight.  1 and 2 peers: 4-wave blocks, <= 8 per CU.  16 peers,
// 4 and 8 in short launches and 4 in large ones: 4-wave blocks <= 4, which spread
// better.  4 and 8 peers otherwise: 8-wave blocks <= 3, or <= 2 for 8 peers with
// chunks of 64 M and more; they suffer less where the chunks of the peers lie a
// large power of two apart (as those of power-of-two widths do) and their rows
// meet in the same memory banks.  8 to 4 bits, 4-wave <= 4 (<= 8 up to 3 peers)
// against 8-wave <= 3:
//   P = 8, chunks of 2^24 29.2 / 26.7, 2^24 + 12288 25.0 / 25.1, 5 * 2^22
//     33.7 / 32.2, 26214400 37.4 / 37.9, 2^19 3.1 / 3.8; 105M and 203M 146.9 /
//     285.6, 8-wave <= 2 140.4 / 277.5
//   P = 4, 2^25 28.4 / 27.1, 2^25 + 12288 26.1 / 26.0; 2^27 101.6 / 103 or more
//   P = 2, 134M 107 / 117;  P = 16, 2^23 28.3 / 29.0, 2^23 + 6144 25.0 / 26.4, 2^24
//     56.3 / 54.2, 11.5M 34.1 / 35.0
// 3, 5 to 7 and 9 to 15 peers: 8-wave blocks <= 3 at every size, for the large
// launches (P = 3 / 6, 64 M 41.6 / 32 M 40.1 and 38.5 / 38.6; 16 M 12.7 / 20.9 and
// 11.5 / 20.5); from 2 to 10 M both shapes are within 5 % either way, and launches
// of 1 M and less are the slower for it (P = 3 / 6, 1 M 2.9 / 3.15 and 3.2 / 3.65).
//
// 4-bit messages: 4-wave blocks, 32 elements per lane (a 16-byte chunk per
// peer) <= 6 per CU for the large launches of up to 7 peers, else 16 per lane
// <= 8, or, from 8 peers and 4 M on, in 8-wave blocks <= 4 (2^29 input
// elements, P = 4 56.3 against 59.7 with 16 per lane; P = 8, chunks of 2^24 /
// 2^24 + 12288 / 50.8M 4-wave 17.8 / 15.0 / 43.7, 8-wave 15.6 / 15.7 / 40.4).
//
// With the float32 copy four fifths and more of a launch's writes are the copy, and
// other shapes serve them better.  4-bit messages of 4 M and more: 1 peer, and up
// to 9 M up to 8 peers, 32 per lane <= 6 (P = 8, 5 M 9.15, 8-wave 16 per lane 10.7);
// 2 to 7 peers then 16 per lane in 4-wave blocks <= 6, for 2 uncapped (P = 4, 11 M 15.3,
// 32 per lane 15.9; P = 6, 12 M 18.1 and 20.3; P = 2, 12 M 12.45, <= 6 13.9) and from 16 M on in 8-wave blocks <= 3 (P = 2 / 4,
// 128 M 114.8 / 138.5, 4-wave 116.5 / 141, 32 per lane 131.9 / 155.9; 1 peer 114.7, 32
// per lane 110.5).  8-bit messages of 16 peers from 4.75 M on: 8-wave blocks <= 3
// (chunks of 5 / 6 / 8 / 16 M 21.8 / 24.8 / 35.6 / 67.5, 4-wave 22.3 / 26.3 / 38.0 /
// 72.5; sizes between within 2 % either way; 4 to 4.6 M 21.9 and 20.0).
//
// Stochastic rounding takes the same shapes.  Its kernels are bound by instructions,
// and a cap does not move them (8 to 4 bits, as here and uncapped: P = 2, 128 M 68.7
// and 68.5; P = 4, 44 M 35.0 and 36.6; P = 8, 32 M 51.7 and 51.5; P = 16, 12 M 40.5
// and 40.3; 4 to 4 bits P = 4, 128 M 79.5 and 76.8, P = 8, 44 M 43.4 and 43.0).
template <int E_, int WPB_, uint32_t PEERS_>
struct Shape { // elements per lane, waves per block, peer counts that take it
    static constexpr int E = E_, WPB = WPB_;
    static constexpr uint32_t PEERS = PEERS_;
};

template <int BITS_IN, int BITS_OUT, bool SR>
int requant_for(const PeerTable &peers, int P, int64_t n, int gs, uint8_t *out_codes, float *out_scales, float *out_f32,
                hipStream_t s, uint64_t seed, uint64_t offset)
{
    // groups beyond a wave tile are shared by the waves of a block
    const auto go = [&](auto shape, int cap, auto guarded) {
        using S = decltype(shape);
        const auto run = [&](auto kernel) {
            return launch_tiles<S::E, S::WPB>(kernel, n, cap, s, peers, P, n, gs, out_codes, out_scales, out_f32, seed,
                                              offset);
        };
        const auto pick = [&](auto wide) {
            using R = Requant<BITS_IN, BITS_OUT, S::E, S::WPB, SR, decltype(wide)::value>;
            if constexpr (decltype(guarded)::value)
                return with_guarded_peers<R::template Kernel, S::PEERS>(P, run);
            else
                return with_peers<R::template Kernel, S::PEERS>(P, run);
        };
        return (1 << gs) > kWave * S::E ? pick(std::true_type{}) : pick(std::false_type{});
    };
    constexpr int64_t M = int64_t(1) << 20;
    const auto shaped = [&](auto f32) {
        constexpr bool F32 = decltype(f32)::value; // the float32 copy: the guarded kernels
        if constexpr (BITS_IN == 4) {
            if (n < 4 * M)
                return go(Shape<16, 4, kAllPeers>{}, 8, f32);
            if constexpr (F32) {
                if (P == 1 || (n <= 9 * M && (P < 8 || (P == 8 && n > 4 * M))))
                    return go(Shape<32, 4, peer_range(1, 8)>{}, 6, f32);
                if (P < 8)
                    return n < 16 * M ? go(Shape<16, 4, kAllPeers>{}, P == 2 ? kUncapped : 6, f32)
                                      : go(Shape<16, 8, peer_range(2, 16)>{}, 3, f32);
                return go(Shape<16, 8, peer_range(2, 16)>{}, 4, f32);
            }
            return P < 8 ? go(Shape<32, 4, peer_range(1, 7)>{}, 6, f32) : go(Shape<16, 8, peer_range(8, 16)>{}, 4, f32);
        } else {
            const bool large = n >= 64 * M, small = n < 8 * M;
            if (P & (P - 1) || (P == 8 && !small) || (P == 4 && !small && !large) || (F32 && P == 16 && n >= 19 * M / 4))
                return go(Shape<16, 8, F32 ? peer_range(3, 16) : peer_range(3, 15)>{}, P == 8 && large ? 2 : 3, f32);
            return go(Shape<16, 4, (1u << 1 | 1u << 2 | 1u << 4 | 1u << 8 | 1u << 16)>{}, P >= 4 ? 4 : 8, f32);
        }
    };
    return out_f32 ? shaped(std::true_type{}) : shaped(std::false_type{});
}

template <int BITS_IN, int NB, int E, int WPB>
struct ReduceToF32 {
    template <int PMAX, bool EXACT>
    struct Kernel {
        static auto get() { return k_reduce_to_f32<BITS_IN, E, NB, PMAX, EXACT, WPB>; }
    };
};

// Bytes that a reduction to float32 reads and writes from which it no longer
// runs within the L2 caches (8 of 4 MB), with a transform of NB points: the more
// arithmetic, the later.
template <int NB>
constexpr int64_t kSpill = int64_t(NB == 0 ? 25 : NB <= 64 ? 31 : NB <= 256 ? 33 : 38) << 20;

// Dequantize-reduce to float32: 16 elements per lane (4 KiB written per wave) in
// general.  us with groups of 128, each pass on other inputs; M = 2^20 elements of
// a chunk, MB = 2^20 bytes read and written.
//
// 8-bit messages in 4-wave blocks, <= 5 per CU for one peer, <= 4 for more (2^29
// input elements, <= 4 / 5 / 6 / 8 per CU: P = 2 243 / 247 / 261 / 281; P = 1 2 to
// 5 % faster at 5).  From kSpill (36 MB for 3 peers) to 49 MB, 3 to 8 peers, 6 and
// more up to 4 M, take the guarded kernels: their loads go out one by one, each
// after its peer's pointer, which the caches serve better there and worse elsewhere
// (guarded and exact without a transform / with 256 points: P = 4, 4 M 5.8 and 6.8 /
// 6.1 and 6.1, 5 M 7.1 and 8.3 / 7.0 and 8.1; P = 5, 4 M 6.7 and 7.9 / 7.0 and 8.1;
// P = 8, 3 M 7.2 and 7.6 / 7.6 and 7.6; P = 3, 6 M 7.6 and 8.8 / 7.0 and 8.7; outside,
// P = 4, 3 M 4.95 and 4.85 / 5.5 and 4.9; P = 8, 4.5 M 11.9 and 10.8 / 12.3 and 11.0).
//
// 4-bit messages:
//   1 and 2 peers: 4-wave blocks, uncapped up to 20 M with at most 256 points (P = 1,
//     12 M, no transform 9.7, <= 5 per CU 11.1; 1024 points, 11 M 11.2, <= 5 10.3),
//     above <= 6 and <= 5 (P = 1, 64 M <= 5 / 6 51.9 / 49.8; 2^29 input elements, P = 2
//     <= 4 / 5 / 6 / 8 216 / 208 / 212 / 242).
//   3 to 8 peers from kSpill (5 MB more for 3) on, without a transform also 2 (11 MB
//     more): 32 elements per lane, 8 KiB written per wave, <= 4 per CU, up to 12 M for
//     2 to 4 peers, 6.5 M for 8 (9 M with 512 points and more) (16 and 32 per lane, no
//     transform: P = 2, 8 M 8.4 and 7.1; P = 4, 5.5 M 8.05 and 5.96; P = 6, 4.5 M 8.0
//     and 6.3; P = 8, 4 M 7.9 and 6.6; 256 points: P = 5, 5.5 M 8.5 and 7.1; below
//     kSpill, 256 points, P = 4, 3.5 M 5.1 and 5.5; P = 4, 2^27 124 and 133).  9 to 15
//     peers the same from 5 M, with a transform 9 to 11 from 6.5 M, to 9 M (P = 11, 7 M,
//     no transform / 256 points 14.4 / 15.3, 8-wave blocks 15.8 / 15.8; 8 M with a
//     transform P = 9 / 11 / 12 / 13 16.0 / 18.1 / 20.6 / 21.9 and 17.6 / 18.5 / 19.3 / 19.7).
//     While the result is of the
//     order of the L2s, 6.5 to 8 M, from 4 peers on without a transform in the guarded
//     form (P = 4, 7.5 M 8.2, exact 9.2; P = 7, 7 M 9.5 and 12.0, 9 M 14.6 and 14.7).
//   8 and more peers beyond that, above 5 M: 8-wave blocks <= 3 (P = 8, 2^24 / 50.8M
//     24.9 / 67.7, 4-wave <= 4 26.9 / 71.4; P = 16, 2^23 20.2 and 24.3; with a transform,
//     P = 9 / 11 / 13 / 16, 5.05 to 5.5 M 11.7 / 13.0 / 14.1 / 15.5, 4-wave 12.2 / 13.8 / 15.3
//     / 16.1, 4.6 to 5 M 11.7 / 12.8 / 14.0 / 15.1 and 10.9 / 12.1 / 13.2 / 14.3).
//   4 peers with chunks of 2^24 and more: 2-wave blocks <= 8, for power-of-two chunks
//     (2^25 / 2^26 36.1 / 65.1, 4-wave <= 4 36.7 / 68.0; others the same either way: 44 M
//     44.5, 96 M 95.4 and 93.5, 203M 191.2 and 190.5).
//   The rest: 4-wave blocks, <= 4 from 4 peers on, <= 5 for 3.
template <int BITS_IN, int NB>
int reduce_to_f32(const PeerTable &peers, int P, int64_t n, int gs, float cn, float out_scale, float *out_f32,
                      hipStream_t s)
{
    const auto go = [&](auto shape, int cap, auto guarded) {
        using S = decltype(shape);
        using R = ReduceToF32<BITS_IN, NB, S::E, S::WPB>;
        const auto run = [&](auto kernel) {
            return launch_tiles<S::E, S::WPB>(kernel, n, cap, s, peers, P, n, gs, cn, out_scale, out_f32);
        };
        if constexpr (decltype(guarded)::value)
            return with_guarded_peers<R::template Kernel, S::PEERS>(P, run);
        else
            return with_peers<R::template Kernel, S::PEERS>(P, run);
    };
    constexpr std::true_type guarded{};
    constexpr std::false_type exact{};
    constexpr int64_t M = int64_t(1) << 20;
    const int64_t bytes = n * (8 * 4 + P * BITS_IN) / 8;
    if constexpr (BITS_IN == 4) {
        const int64_t from = kSpill<NB> + (P == 2 ? 11 * M : P == 3 ? 5 * M : 0);
        if (P >= (NB == 0 ? 2 : 3) && (P <= 8 ? bytes >= from : P < (NB == 0 ? 16 : 12) && n > (NB == 0 ? 5 * M : 13 * M / 2))) {
            if constexpr (NB == 0) {
                if (P >= 4 && P <= 8 && n >= 13 * M / 2 && n <= 8 * M)
                    return go(Shape<32, 4, peer_range(4, 8)>{}, 4, guarded);
            }
            if (P <= 4 ? n < 12 * M : P < 8 || (P == 8 ? n < (NB > 256 ? 9 * M : 13 * M / 2) : n <= 9 * M))
                return go(Shape<32, 4, peer_range(NB == 0 ? 2 : 3, 15)>{}, 4, exact);
        }
        if (P >= 8 && n > 5 * M)
            return go(Shape<16, 8, peer_range(8, 16)>{}, 3, exact);
        if (P == 4 && n >= 16 * M)
            return go(Shape<16, 2, 1u << 4>{}, 8, exact);
        return go(Shape<16, 4, kAllPeers>{},
                  P >= 4 ? 4 : P == 3 ? 5 : NB <= 256 && n <= 20 * M ? kUncapped : P == 1 ? 6 : 5, exact);
    } else {
        if (P >= 3 && P <= 8 && bytes >= (P == 3 ? 36 * M : kSpill<NB>) && bytes <= 49 * M && (P <= 5 || n <= 4 * M))
            return go(Shape<16, 4, peer_range(3, 8)>{}, 4, guarded);
        return go(Shape<16, 4, kAllPeers>{}, P >= 2 ? 4 : 5, exact);
    }
}

} // namespace sdp4
