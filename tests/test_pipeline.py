"""HotPath's host logic: which chunks its reductions are given."""
import pytest

torch = pytest.importorskip("torch")

from paper_2410_15526_amd import sdp4  # noqa: E402
from paper_2410_15526_amd.pipeline import HotPath  # noqa: E402


@pytest.fixture
def calls(monkeypatch):
    """The chunks of each reduction, with addresses offered for every plain buffer; nothing is launched."""
    got = []
    monkeypatch.setattr(sdp4, "chunk_addresses", lambda *a: (["addresses"], ["addresses"]))
    for name in ("sdp4_dequant_reduce", "sdp4_dequant_reduce_sr"):
        monkeypatch.setattr(sdp4, name, lambda codes, scales, *a, **k: got.append((codes, scales)))
    return got


def reductions(h):
    h.reduce_intra()
    h.reduce_inter()
    h.reduce_intra_sr()


def make(cls):
    return cls(1 << 14, 64, 64, 4, 2, 128, "f32", device="cpu")


def test_own_buffers_go_by_address(calls):
    reductions(make(HotPath))
    assert calls == [(["addresses"], ["addresses"])] * 3


def test_chunks_of_a_subclass_are_used(calls):
    class Received(HotPath):
        def intra_chunks(self, bits=8):
            return ["c8"] * self.P, ["s8"] * self.P

        def inter_chunks(self):
            return ["c4"] * self.Q, ["s4"] * self.Q

    reductions(make(Received))
    assert calls == [(["c8"] * 4, ["s8"] * 4), (["c4"] * 2, ["s4"] * 2), (["c8"] * 4, ["s8"] * 4)]


def test_chunks_set_on_an_object_are_used(calls):
    h = make(HotPath)
    h.intra_chunks = lambda bits=8: ("c8", "s8")
    h.inter_chunks = lambda: ("c4", "s4")
    reductions(h)
    assert calls == [("c8", "s8"), ("c4", "s4"), ("c8", "s8")]


def test_chunks_of_another_object_are_used(calls):
    """Bound methods of another HotPath, whose message is the one to reduce."""
    h, other = make(HotPath), make(HotPath)
    h.intra_chunks, h.inter_chunks = other.intra_chunks, other.inter_chunks
    reductions(h)
    buffers = [other.c8, other.c4, other.c8]
    assert [c[0][0].data_ptr() for c in calls] == [b.data_ptr() for b in buffers]


def test_chunks_patched_into_the_class_are_used(calls, monkeypatch):
    monkeypatch.setattr(HotPath, "intra_chunks", lambda self, bits=8: ("c8", "s8"))
    monkeypatch.setattr(HotPath, "inter_chunks", lambda self: ("c4", "s4"))
    reductions(make(HotPath))
    assert calls == [("c8", "s8"), ("c4", "s4"), ("c8", "s8")]
