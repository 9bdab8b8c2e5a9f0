"""The binding's native marshalling against its general path: what it takes
over, what it leaves alone, and that nothing is called for what it leaves."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")

from paper_2410_15526_amd import sdp4  # noqa: E402
from tests._gpu import empty  # noqa: E402


def native():
    sdp4.lib()
    assert sdp4._fast is not None
    return sdp4._fast


N, G = 4096, 128


def _unbound(monkeypatch):
    """sdp4 as before its first call, to be put back after the test."""
    native()
    monkeypatch.setattr(sdp4, "_lib", None)
    monkeypatch.setattr(sdp4, "_fast", None)


def _takes_the_general_path():
    L = sdp4.lib()
    assert sdp4._fast is None and sdp4.sdp4_num_groups(N, G) == N // G
    assert sdp4.chunk_addresses(None, None, 1, 0, 0) is None
    with pytest.raises(sdp4.Sdp4Error) as e:                                      # an unknown code width, no HIP call
        sdp4.sdp4_grad_quant(1 << 20, 5, 0, G, 1 << 21, 1 << 22, N, 0)
    assert e.value.status == sdp4.EINVAL and L is sdp4.lib()


@pytest.mark.cpu_only
def test_library_without_its_binding_says_so_and_works(monkeypatch):
    import sys

    import paper_2410_15526_amd as package
    _unbound(monkeypatch)
    monkeypatch.delattr(package, "_binding")
    monkeypatch.setitem(sys.modules, "paper_2410_15526_amd._binding", None)       # its import raises ImportError
    with pytest.warns(RuntimeWarning, match="no native argument marshalling"):
        _takes_the_general_path()


@pytest.mark.cpu_only
def test_binding_of_another_torch_is_not_used(monkeypatch):
    f = native()
    assert f.torch_version == torch.__version__
    _unbound(monkeypatch)
    monkeypatch.setattr(f, "torch_version", "1.0")
    with pytest.warns(RuntimeWarning, match="built for torch 1.0"):
        _takes_the_general_path()


@pytest.mark.cpu_only
def test_binding_that_does_not_name_its_torch_is_not_used(monkeypatch):
    """One built from sources that recorded no version."""
    f = native()
    _unbound(monkeypatch)
    monkeypatch.delattr(f, "torch_version")
    with pytest.warns(RuntimeWarning, match="built for torch None"):
        _takes_the_general_path()


@pytest.mark.cpu_only
def test_leaves_what_is_not_on_a_gpu_or_not_ordinary():
    f = native()
    t = lambda n, dt=torch.float32: torch.zeros(n, dtype=dt)  # noqa: E731
    w, q, h = t(N), t(N // 2, torch.uint8), t(N // G)
    assert f.qwd_encode(w, w, G, q, h, h, None, None) is None                     # host tensors
    assert f.qwd_encode(object(), w, G, q, h, h, None, None) is None
    assert f.qwd_encode(w, w, G, q, h, h, None) is None                           # too few arguments
    assert f.qwd_encode(4096, 8192, G, 16, 32, 48, 1.5, None) is None
    assert f.qwd_encode(4096, 8192, True, 16, 32, 48, N, 0) is None               # not a plain int
    assert f.grad_quant(1 << 20, 5.0, 0, G, 1 << 21, 1 << 22, N, 0) is None
    assert f.grad_quant(1 << 200, 8, 0, G, 1 << 21, 1 << 22, N, 0) is None        # not an address
    assert f.grad_quant(1 << 20, 8, 0, G, 1 << 21, 1 << 22, 1 << 60, 0) is None   # beyond the element limit
    assert f.dequant_reduce([1 << 20] * 17, [1 << 21] * 17, N, 8, G, 4, 0, 1.0, 1, 2, None, 0) is None
    assert f.dequant_reduce([1 << 20] * 2, [1 << 21] * 3, N, 8, G, 4, 0, 1.0, 1, 2, None, 0) is None
    assert f.chunk_addresses(q, h, 4, 16, 1) is None
    with pytest.raises(ValueError, match="device tensors"):
        sdp4.sdp4_qwd_encode(w, w, G, q, h, h)


@pytest.mark.cpu_only
def test_statuses_come_back_as_from_the_general_path():
    """Addresses that the library rejects before any HIP call, both ways."""
    f, L = native(), sdp4.lib()
    for bits, block, group, n, x in ((8, 3, G, N, 1 << 20), (8, 0, 100, N, 1 << 20), (8, 0, G, N + 1, 1 << 20),
                                     (8, 0, G, N, (1 << 20) + 4), (4, 0, G, 0, 1 << 20)):
        got = f.grad_quant(x, bits, block, group, 1 << 21, 1 << 22, n, 0)
        assert got == L.sdp4_grad_quant(x, n, bits, block, group, 1 << 21, 1 << 22, None)
    with pytest.raises(sdp4.Sdp4Error) as e:
        sdp4.sdp4_grad_quant(1 << 20, 8, 3, G, 1 << 21, 1 << 22, n=N, stream=0)
    assert e.value.status == sdp4.EINVAL
    cp, sp = (C.c_void_p * 2)(1 << 20, 1 << 21), (C.c_void_p * 2)(1 << 22, 1 << 23)
    for out_scale, P in ((float("inf"), 2), (1.0, 0)):
        got = f.dequant_reduce([1 << 20, 1 << 21][:P], [1 << 22, 1 << 23][:P], N, 8, G, 0, 0, out_scale, None, None,
                               1 << 24, 0)
        assert got == L.sdp4_dequant_reduce(P, cp, sp, N, 8, G, 0, 0, out_scale, None, None, 1 << 24, None) != 0


@pytest.mark.gpu
@pytest.mark.parametrize("stream", ["current", "other", "address"])
def test_same_results_as_the_general_path(stream, monkeypatch):
    torch.manual_seed(1)
    g = torch.Generator(device="cuda").manual_seed(3)
    prev = torch.randn(N, device="cuda", generator=g).to(torch.bfloat16)
    new = prev.float() + 1e-3 * torch.randn(N, device="cuda", generator=g)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    arg = {"current": None, "other": side, "address": side.cuda_stream}[stream]

    def once():
        w = prev.clone()
        q, s, m = empty(N // 2, "u8"), empty(N // G, "f32"), empty(N // G, "f32")
        c8, s8 = empty(N, "u8"), empty(N // G, "f32")
        c4, s4, out = empty(N // 8, "u8"), empty(N // 4 // G, "f32"), empty(N // 4, "f32")
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            sdp4.sdp4_qwd_encode(new, w, G, q, s, m, stream=arg)
            sdp4.sdp4_qwd_decode(q, s, m, G, w, stream=arg)
            sdp4.sdp4_grad_quant(new, 8, 64, G, c8, s8, stream=arg)
            sdp4.sdp4_dequant_reduce(c8.chunk(4), s8.chunk(4), N // 4, 8, G, 4, out_codes=c4, out_scales=s4, stream=arg)
            sdp4.sdp4_dequant_reduce([c4], [s4], N // 4, 4, G, 0, 64, 0.25, out_f32=out, stream=arg)
        torch.cuda.synchronize()
        return q, s, m, w, c8, s8, c4, s4, out

    native()
    a = once()
    monkeypatch.setattr(sdp4, "_fast", None)
    b = once()
    assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.gpu
def test_refuses_short_strided_and_mistyped_tensors():
    native()
    x, s = torch.zeros(N, device="cuda"), empty(N // G, "f32")
    with pytest.raises(ValueError, match="codes"):
        sdp4.sdp4_grad_quant(x, 8, 0, G, empty(N - 1, "u8"), s)
    with pytest.raises(ValueError, match="contiguous"):
        sdp4.sdp4_grad_quant(torch.zeros(2 * N, device="cuda")[::2], 8, 0, G, empty(N, "u8"), s)
    with pytest.raises(ValueError, match="float32 or bfloat16"):
        sdp4.sdp4_qwd_encode(x, x.half(), G, empty(N // 2, "u8"), s, s.clone())
    assert sdp4.chunk_addresses(empty(N, "u8"), s, 4, N // 4 + 1, 8) is None
    c, h = sdp4.chunk_addresses(x.view(torch.uint8), s, 4, N // 4, N // 4 // G)
    assert c == [x.data_ptr() + i * N // 4 for i in range(4)] and h == [s.data_ptr() + 32 * i for i in range(4)]
