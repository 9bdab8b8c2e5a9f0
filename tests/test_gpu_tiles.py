"""GPU parity at the places where the kernels' code paths change: the edges
of lane slices, tiles and blocks, and the choices of the launchers.  All
results are compared with the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2410_15526_amd import sdp4
from tests._gpu import check_f32, dev, empty, host, say, torch

pytestmark = pytest.mark.gpu


def sync():
    torch().cuda.synchronize()


@pytest.mark.parametrize("P", [1, 3, 4])
def test_every_nibble_at_every_position_with_extreme_scales(P):
    """4-bit codes become floats exactly, also under denormal and huge scales."""
    group, n = 32, 32 * 64
    say(f"nibbles P={P}")
    q = np.stack([np.roll(np.arange(16, dtype=np.uint8), r) for r in range(16)]).reshape(-1)   # 16 x 16
    q = np.resize(q, n)
    codes = (q[0::2] | (q[1::2] << 4)).astype(np.uint8)
    scales = np.resize(np.float32([1e-45, 3e-41, 1.2e-38, 1e-30, 0.1, 1.0, 3e7, 1e36]), n // group)
    msgs = [(np.roll(codes, p), np.roll(scales, p)) for p in range(P)]
    out = empty(n, "f32")
    sdp4.sdp4_dequant_reduce([dev(c) for c, _ in msgs], [dev(s) for _, s in msgs], n, 4, group, 0, 0, 1.0, None, None, out)
    sync()
    ref = oracle.dequant_reduce([c for c, _ in msgs], [s for _, s in msgs], n, 4, group, 0, 0, 1.0)
    check_f32(host(out), ref["f32"])


def _weights(n, bf16, seed):
    rng = np.random.default_rng(seed)
    prev = rng.standard_normal(n, dtype=np.float32) * np.float32(0.02)
    if bf16:
        prev = oracle.bf16_rne(prev)
    wide = oracle.bf16_to_f32(prev) if bf16 else prev
    return wide + rng.standard_normal(n, dtype=np.float32) * np.float32(5e-4), prev


# One group, one block (2048 and 4096 elements), one group less or more, and
# several blocks with a partial last one; groups inside a wave tile (512, 1024
# elements), over it, and as large as a block.
SIZES = [(32, 32), (32, 2048 - 32), (32, 4096 + 32), (512, 4096 - 512), (512, 3 * 4096 + 512), (1024, 1024),
         (1024, 5 * 4096 - 1024), (2048, 2048), (2048, 4096), (2048, 3 * 4096 + 2048), (4096, 4096), (4096, 5 * 4096)]


@pytest.mark.parametrize("group,n", SIZES)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("sym", [False, True])
def test_qwd_at_block_edges(group, n, bf16, sym):
    say(f"qwd edges group={group} n={n} bf16={bf16} sym={sym}")
    new, prev = _weights(n, bf16, n + group)
    pd = dev(prev)
    codes, scale, minv = empty(n // 2, "u8"), empty(n // group, "f32"), empty(n // group, "f32")
    if sym:
        sdp4.sdp4_qwd_encode_sym(dev(new), pd, group, codes, scale)
        want = oracle.qwd_encode_sym(new, prev, group)
        sdp4.sdp4_qwd_decode_sym(codes, scale, group, pd)
        after = oracle.qwd_decode_sym(want[0], want[1], prev, group)
    else:
        sdp4.sdp4_qwd_encode(dev(new), pd, group, codes, scale, minv)
        want = oracle.qwd_encode(new, prev, group)
        sdp4.sdp4_qwd_decode(codes, scale, minv, group, pd)
        after = oracle.qwd_decode(want[0], want[1], want[2], prev, group)
        assert np.array_equal(host(minv), want[2])
    sync()
    assert np.array_equal(host(codes), want[0]) and np.array_equal(host(scale), want[1])
    assert np.array_equal(host(pd), after)


@pytest.mark.parametrize("group,n", SIZES)
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("block", [0, 32, 512])
@pytest.mark.parametrize("sr", [False, True])
def test_grad_quant_at_block_edges(group, n, bits, block, sr):
    n = -(-n // max(block, 1)) * max(block, 1)
    say(f"grad_quant edges group={group} n={n} bits={bits} block={block} sr={sr}")
    x = np.random.default_rng(n + bits).standard_normal(n, dtype=np.float32) * np.float32(1e-4)
    codes, scale = empty(n * bits // 8, "u8"), empty(n // group, "f32")
    if sr:
        sdp4.sdp4_grad_quant_sr(dev(x), bits, block, group, 77, 8, codes, scale)
        want = oracle.grad_quant_sr(x, bits, block, group, 77, 8)
    else:
        sdp4.sdp4_grad_quant(dev(x), bits, block, group, codes, scale)
        want = oracle.grad_quant(x, bits, block, group)
    sync()
    assert np.array_equal(host(codes), np.ascontiguousarray(want[0]).view(np.uint8))
    assert np.array_equal(host(scale), want[1])


def _messages(P, n, bits, group, seed):
    rng = np.random.default_rng(seed)
    top = 127 if bits == 8 else 7
    out = []
    for _ in range(P):
        q = np.clip(np.rint(rng.standard_normal(n, dtype=np.float32) * (top / 3)), -top, top).astype(np.int8)
        codes = q.view(np.uint8) if bits == 8 else ((q[0::2] & 15) | ((q[1::2] & 15) << 4)).astype(np.uint8)
        out.append((codes, (np.exp(rng.standard_normal(n // group)) * 1e-5).astype(np.float32)))
    return out


# Every peer count with a kernel of its own and one of each guarded kernel,
# at block edges of the shapes of small launches.
@pytest.mark.parametrize("P", [1, 2, 3, 4, 5, 8, 11, 16])
@pytest.mark.parametrize("bits_in", [4, 8])
@pytest.mark.parametrize("group,n", [(32, 4096 + 32), (1024, 3 * 4096 - 1024), (2048, 8192 + 2048), (4096, 8192 + 4096)])
def test_requant_at_block_edges(P, bits_in, group, n):
    say(f"requant edges P={P} in={bits_in} group={group} n={n}")
    msgs = _messages(P, n, bits_in, group, P + n)
    cd, sd = [dev(c) for c, _ in msgs], [dev(s) for _, s in msgs]
    for bits_out in (4, 8):
        for seed in (None, 5):
            oc, osc = empty(n * bits_out // 8, "u8"), empty(n // group, "f32")
            if seed is None:
                sdp4.sdp4_dequant_reduce(cd, sd, n, bits_in, group, bits_out, out_codes=oc, out_scales=osc)
                ref = oracle.dequant_reduce([c for c, _ in msgs], [s for _, s in msgs], n, bits_in, group, bits_out)
            else:
                sdp4.sdp4_dequant_reduce_sr(cd, sd, n, bits_in, group, bits_out, seed, 16, oc, osc)
                ref = oracle.dequant_reduce_sr([c for c, _ in msgs], [s for _, s in msgs], n, bits_in, group, bits_out,
                                               seed, 16)
            sync()
            assert np.array_equal(host(oc), np.ascontiguousarray(ref["codes"]).view(np.uint8))
            assert np.array_equal(host(osc), ref["scales"])


@pytest.mark.parametrize("group,extra", [(128, -128), (128, 0), (128, 128), (2048, 2048), (4096, 4096)])
def test_requant_of_4_bit_messages_around_its_lane_width_switch(group, extra):
    P, n = 3, (1 << 22) + extra
    say(f"requant 4-bit n={n} group={group}")
    msgs = _messages(P, n, 4, group, n)
    oc, osc = empty(n // 2, "u8"), empty(n // group, "f32")
    sdp4.sdp4_dequant_reduce([dev(c) for c, _ in msgs], [dev(s) for _, s in msgs], n, 4, group, 4, out_codes=oc,
                             out_scales=osc)
    sync()
    ref = oracle.dequant_reduce([c for c, _ in msgs], [s for _, s in msgs], n, 4, group, 4)
    assert np.array_equal(host(oc), np.ascontiguousarray(ref["codes"]).view(np.uint8))
    assert np.array_equal(host(osc), ref["scales"])


def test_launch_of_more_blocks_than_one_grid_dimension_takes():
    """2^22 blocks go along x: a decode of more than 2^32 float32 weights (1024
    per block) covers a second row.  Scales, minima and weights are small whole
    numbers, so every result is exact in float32."""
    t = torch()
    group, n = 4096, (1 << 32) + 5 * 4096
    say(f"decode n={n}")
    w = t.ones(n, dtype=t.float32, device="cuda")
    codes = t.randint(0, 256, (n // 2,), dtype=t.uint8, device="cuda")
    scale = t.randint(1, 8, (n // group,), device="cuda").float()
    minv = t.randint(-8, 8, (n // group,), device="cuda").float()
    sdp4.sdp4_qwd_decode(codes, scale, minv, group, w)
    for a, b in ((0, 1 << 20), ((1 << 32) - (1 << 20), (1 << 32) + 4096), (n - 4096, n)):
        c = codes[a // 2:b // 2]
        q = t.stack((c & 15, c >> 4), 1).view(-1, group).float()
        want = 1 + q * scale[a // group:b // group].view(-1, 1) + minv[a // group:b // group].view(-1, 1)
        assert t.equal(w[a:b].view(-1, group), want), (a, b)


@pytest.mark.parametrize("bits", [4, 8])
def test_stochastic_rounding_of_group_extremes(bits):
    """Elements at +-(the group's largest magnitude), whose product with the
    inverse scale can land one ulp beyond the last level, on either side."""
    group, groups = 32, 1 << 14
    say(f"sr extremes bits={bits}")
    rng = np.random.default_rng(bits)
    s = np.exp(rng.uniform(-60, 60, groups)).astype(np.float32)
    x = (rng.choice(np.float32([-1, 1]), (groups, group)) * s[:, None]).astype(np.float32).reshape(-1)
    codes, scale = empty(x.size * bits // 8, "u8"), empty(groups, "f32")
    for seed in range(3):
        sdp4.sdp4_grad_quant_sr(dev(x), bits, 0, group, seed, 0, codes, scale)
        sync()
        want = oracle.grad_quant_sr(x, bits, 0, group, seed, 0)
        assert np.array_equal(host(codes), np.ascontiguousarray(want[0]).view(np.uint8))
        assert np.array_equal(host(scale), want[1])


@pytest.mark.parametrize("bits,top", [(8, 127.0), (4, 7.0)])
def test_stochastic_rounding_of_negative_denormals(bits, top):
    """A product that is a negative denormal rounds down to -1 where the uniform is 0 (17 of these elements), and
    would to 0 if the conversion flushed it."""
    group, n = 32, 1 << 20
    say(f"sr denormals bits={bits}")
    x = np.full(n, -1e-41, np.float32)
    x[::group] = top                                                       # inverse scale 1
    codes, scale = empty(n * bits // 8, "u8"), empty(n // group, "f32")
    sdp4.sdp4_grad_quant_sr(dev(x), bits, 0, group, 0, 0, codes, scale)
    sync()
    want = oracle.grad_quant_sr(x, bits, 0, group, 0, 0)
    w = np.ascontiguousarray(want[0]).view(np.uint8)
    assert np.sum(w == 0xFF) + (np.sum(w & 15 == 15) + np.sum(w >> 4 == 15) if bits == 4 else 0) == 17
    assert np.array_equal(host(codes), w) and np.array_equal(host(scale), want[1])


@pytest.mark.parametrize("bits,block,group,n", [
    (b, blk, 512, (1 << 25) + extra) for b, blk in ((8, 256), (4, 0), (4, 128), (4, 256)) for extra in (-512, 512)] + [
    # 4 to 9 times 2^20 elements, and 4-bit codes in groups of 1024 and more below 2^25
    (4, 0, 512, 1 << 22), (4, 0, 32, (1 << 22) + 32), (8, 256, 512, 9 << 20), (8, 32, 64, (9 << 20) + 64),
    (8, 128, 4096, (1 << 22) + 4096), (8, 64, 1024, 9 << 20), (4, 16, 32, 5 << 20), (4, 2, 2048, (1 << 22) + 2048),
    (4, 0, 2048, (1 << 25) - 2048), (4, 0, 2048, 1 << 25), (4, 64, 1024, (9 << 20) + 1024)])
def test_grad_quant_around_its_block_shape_switches(bits, block, group, n):
    say(f"grad_quant bits={bits} block={block} group={group} n={n}")
    x = np.random.default_rng(bits).standard_normal(n, dtype=np.float32)
    codes, scale = empty(n * bits // 8, "u8"), empty(n // group, "f32")
    sdp4.sdp4_grad_quant(dev(x), bits, block, group, codes, scale)
    sync()
    want = oracle.grad_quant(x, bits, block, group)
    assert np.array_equal(host(codes), np.ascontiguousarray(want[0]).view(np.uint8))
    assert np.array_equal(host(scale), want[1])


@pytest.mark.parametrize("group,n", [(128, 1 << 27), (1024, (1 << 27) + 1024), (2048, (1 << 28) - 2048),
                                     (2048, (1 << 28) + 2048)])
def test_bf16_encode_at_its_block_shape_switches(group, n):
    say(f"encode bf16 n={n} group={group}")
    new, prev = _weights(1 << 20, True, group)
    reps = n // (1 << 20) + 1
    new_d, prev_d = dev(new).repeat(reps)[:n].clone(), dev(prev).repeat(reps)[:n].clone()
    codes, scale, minv = empty(n // 2, "u8"), empty(n // group, "f32"), empty(n // group, "f32")
    sdp4.sdp4_qwd_encode(new_d, prev_d, group, codes, scale, minv)
    want = [dev(a) for a in oracle.qwd_encode(new, prev, group)[:3]]
    t = torch()
    for got, w in zip((codes, scale, minv), want):
        assert t.equal(got, w.repeat(reps)[:got.numel()])


def test_requant_of_8_peers_at_its_block_shape_switch():
    """Chunks of 2^26 elements and one group more; the peers share one message."""
    group, n = 4096, (1 << 26) + 4096
    say(f"requant P=8 n={n}")
    (c, s), = _messages(1, 1 << 20, 8, group, 9)
    reps = n // (1 << 20) + 1
    cd, sd = dev(c).repeat(reps)[:n].clone(), dev(s).repeat(reps)[:n // group].clone()
    want = oracle.dequant_reduce([c] * 8, [s] * 8, 1 << 20, 8, group, 4)
    wc, ws = dev(np.ascontiguousarray(want["codes"]).view(np.uint8)), dev(want["scales"])
    t = torch()
    for m in (n - 4096, n):
        oc, osc = empty(m // 2, "u8"), empty(m // group, "f32")
        sdp4.sdp4_dequant_reduce([cd] * 8, [sd] * 8, m, 8, group, 4, out_codes=oc, out_scales=osc)
        assert t.equal(oc, wc.repeat(reps)[:m // 2]) and t.equal(osc, ws.repeat(reps)[:m // group])


M = 1 << 20


# Above 4 M elements 4-bit messages of up to 7 peers take 32 elements per lane, of more peers 8-wave blocks; with
# the float32 copy shapes of their own.  Each size on either side of a switch, with a partial last block.
@pytest.mark.parametrize("bits_in,P,n", [(4, 1, 4 * M), (4, 3, 4 * M + 8192), (4, 4, 9 * M - 4096), (4, 4, 9 * M),
                                         (4, 7, 16 * M - 4096), (4, 2, 16 * M), (4, 8, 4 * M), (4, 8, 4 * M + 4096),
                                         (4, 8, 9 * M), (4, 11, 4 * M + 4096), (4, 16, 4 * M), (8, 16, 4 * M - 4096),
                                         (8, 16, 4 * M), (8, 16, 19 * M // 4 - 8192),
                                         (8, 16, 19 * M // 4 - 4096), (8, 11, 4 * M + 4096), (8, 5, 12288), (8, 8, 8 * M + 4096)])
@pytest.mark.parametrize("group", [32, 4096])
def test_large_requant_with_and_without_the_float32_copy(bits_in, P, n, group):
    n += group
    say(f"requant with copy P={P} in={bits_in} group={group} n={n}")
    codes, scales = _messages(1, M, bits_in, group, P + n)[0]
    c = [np.resize(np.roll(codes, 16 * group * p), n * bits_in // 8) for p in range(P)]
    s = [np.resize(np.roll(scales, p), n // group) for p in range(P)]
    cd, sd = [dev(x) for x in c], [dev(x) for x in s]
    for bits_out in (4, 8):
        for seed in (None, 5):
            if seed is None:
                ref = oracle.dequant_reduce(c, s, n, bits_in, group, bits_out)
            else:
                ref = oracle.dequant_reduce_sr(c, s, n, bits_in, group, bits_out, seed, 16)
            for copy in (False, True):
                oc, osc = empty(n * bits_out // 8, "u8"), empty(n // group, "f32")
                out = empty(n, "f32") if copy else None
                if seed is None:
                    sdp4.sdp4_dequant_reduce(cd, sd, n, bits_in, group, bits_out, out_codes=oc, out_scales=osc, out_f32=out)
                else:
                    sdp4.sdp4_dequant_reduce_sr(cd, sd, n, bits_in, group, bits_out, seed, 16, oc, osc, out)
                sync()
                assert np.array_equal(host(oc), np.ascontiguousarray(ref["codes"]).view(np.uint8))
                assert np.array_equal(host(osc), ref["scales"])
                if copy:
                    check_f32(host(out), ref["f32"])


# Chunk sizes on either side of every switch of the float32 reductions, most of them bytes read and written
# (25, 31, 33 or 38 MB by the transform's points), with and without a transform that spans lanes.
F32_4_BIT = [(0, 4, 4368896), (0, 4, 4369152), (0, 4, 13 * M // 2 - 256), (0, 4, 13 * M // 2), (0, 7, 8 * M),
             (0, 7, 8 * M + 256), (0, 8, 25 * M // 8 - 256), (0, 8, 25 * M // 8), (0, 8, 13 * M // 2), (0, 8, 8 * M + 256),
             (0, 3, 5719552), (0, 3, 5719808), (0, 3, 12 * M), (0, 11, 5 * M), (0, 11, 5 * M + 256), (0, 9, 9 * M + 256),
             (0, 16, 5 * M), (0, 16, 5 * M + 256), (256, 11, 5 * M), (256, 11, 5 * M + 256),
             (0, 16, 6 * M - 256), (0, 16, 6 * M), (0, 2, 20 * M), (0, 1, 20 * M + 256), (32, 5, 5000960), (32, 5, 5001216),
             (0, 2, 36 * M // 5), (0, 2, 36 * M // 5 + 256), (0, 2, 12 * M), (64, 6, 6 * M), (256, 7, 4613632), (256, 7, 4613888), (256, 4, 12 * M - 256), (256, 4, 12 * M),
             (256, 4, 16 * M - 256), (256, 4, 16 * M), (256, 8, 13 * M // 2 - 256), (256, 8, 13 * M // 2),
             (256, 11, 13 * M // 2 + 256), (256, 12, 7 * M), (2, 4, 7 * M), (512, 6, 6 * M), (1024, 6, 5691392), (1024, 6, 5692416),
             (1024, 1, 11 * M), (1024, 8, 7 * M), (512, 8, 9 * M)]
F32_8_BIT = [(0, 4, 25 * M // 8 - 256), (0, 4, 25 * M // 8), (0, 4, 49 * M // 8), (0, 4, 49 * M // 8 + 256), (0, 3, 5392896),
             (0, 3, 5393152), (0, 8, 4 * M), (0, 8, 4 * M + 256), (256, 5, 4 * M), (1024, 5, 38 * M // 8), (32, 6, 13 * M // 4)]


@pytest.mark.parametrize("bits,block,P,n", [(4, *c) for c in F32_4_BIT] + [(8, *c) for c in F32_8_BIT])
def test_reduction_to_f32_around_its_shape_switches(bits, block, P, n):
    group = 32 if block == 2 else 128
    n = n // max(block, group) * max(block, group)
    say(f"reduce f32 bits={bits} P={P} n={n} group={group} block={block}")
    codes, scales = _messages(1, M, bits, group, P + n)[0]
    c = [np.resize(np.roll(codes, 16 * group * p), n * bits // 8) for p in range(P)]
    s = [np.resize(np.roll(scales, p), n // group) for p in range(P)]
    out = empty(n, "f32")
    sdp4.sdp4_dequant_reduce([dev(x) for x in c], [dev(x) for x in s], n, bits, group, 0, block, 0.25, out_f32=out)
    sync()
    ref = oracle.dequant_reduce(c, s, n, bits, group, 0, block, 0.25)
    check_f32(host(out), ref["f32"])


@pytest.mark.parametrize("P,n", [(4, 1 << 23), (8, (1 << 23) - 4096), (8, 1 << 23), (5, 3 << 12), (16, 1 << 22)])
@pytest.mark.parametrize("bits_in", [4, 8])
def test_requant_around_its_block_shape_switches(P, n, bits_in):
    group = 4096
    say(f"requant P={P} n={n} bits={bits_in}")
    msgs = _messages(1, min(n, 1 << 20), bits_in, group, P)
    c = [np.resize(np.roll(msgs[0][0], 16 * p), n * bits_in // 8) for p in range(P)]
    s = [np.resize(np.roll(msgs[0][1], p), n // group) for p in range(P)]
    oc, osc = empty(n // 2, "u8"), empty(n // group, "f32")
    sdp4.sdp4_dequant_reduce([dev(x) for x in c], [dev(x) for x in s], n, bits_in, group, 4, out_codes=oc, out_scales=osc)
    sync()
    ref = oracle.dequant_reduce(c, s, n, bits_in, group, 4)
    assert np.array_equal(host(oc), np.ascontiguousarray(ref["codes"]).view(np.uint8))
    assert np.array_equal(host(osc), ref["scales"])
