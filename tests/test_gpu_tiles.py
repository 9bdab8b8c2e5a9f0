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
