"""The build's host logic: what it needs and what it leaves out."""
import os
import sys

import pytest

from paper_2410_15526_amd import build


@pytest.fixture
def small(tmp_path, monkeypatch):
    """The build of the two host sources alone, into a folder of its own."""
    monkeypatch.setattr(build, "SOURCES", ["launch.cpp", "abi.cpp"])
    monkeypatch.setattr(build, "BUILD", str(tmp_path / "obj"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libsdp4.so"))
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    return tmp_path


def test_library_builds_without_torch(small, monkeypatch):
    monkeypatch.setitem(sys.modules, "torch", None)          # import torch raises ImportError
    assert build.build() == str(small / "libsdp4.so")
    assert os.path.getsize(small / "libsdp4.so") > 0 and not os.path.exists(small / "_binding.so")


def test_library_builds_beside_a_torch_without_rocm(small, monkeypatch):
    torch = pytest.importorskip("torch")
    monkeypatch.setattr(torch.version, "hip", None)
    build.build()
    assert os.path.getsize(small / "libsdp4.so") > 0 and not os.path.exists(small / "_binding.so")


def test_library_is_there_when_the_binding_does_not_compile(small, monkeypatch):
    def fails(out):
        raise RuntimeError("g++ failed for binding.cpp")
    monkeypatch.setattr(build, "build_binding", fails)
    with pytest.raises(RuntimeError, match="binding.cpp"):
        build.build()
    assert os.path.getsize(small / "libsdp4.so") > 0
