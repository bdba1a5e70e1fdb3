"""The library without the C++ module of its binding: it is built where there is no torch, and without the module every call goes
through ctypes."""
import ctypes
import os
import sys

import pytest
import torch

from paper_2605_24058_amd import binding


def test_the_library_is_built_without_torch(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_SOURCES", ("lordba_pack.cpp",))   # (one unit: what is tried is the build, not the kernels)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "liblordba.so"))
    monkeypatch.setattr(binding, "_TORCH_MODULE_PATH", str(tmp_path / "_lordba_torch.so"))
    monkeypatch.setitem(sys.modules, "torch", None)
    assert binding.build_library() == str(tmp_path / "liblordba.so")
    assert os.listdir(tmp_path) == ["liblordba.so"]
    lib = ctypes.CDLL(str(tmp_path / "liblordba.so"))
    lib.lordba_packed_words.restype, lib.lordba_packed_words.argtypes = ctypes.c_size_t, [ctypes.c_int64] * 2
    assert lib.lordba_packed_words(3, 11) == 2


def test_a_module_that_does_not_compile_leaves_a_library(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_SOURCES", ("lordba_pack.cpp",))
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "liblordba.so"))
    monkeypatch.setattr(binding, "_torch_module_command", lambda tag: (str(tmp_path / "m.o"), [sys.executable, "-c", "print('no such header'); exit(1)"]))
    with pytest.raises(RuntimeError, match="its torch module is not(.|\n)*no such header"):
        binding.build_library()
    assert os.listdir(tmp_path) == ["liblordba.so"]


def _without_module(monkeypatch):
    monkeypatch.setattr(binding, "_torch_module", None)
    monkeypatch.setitem(sys.modules, "paper_2605_24058_amd._lordba_torch", None)   # (its import fails)


def test_calls_without_the_module_are_checked_by_the_binding(monkeypatch):
    _without_module(monkeypatch)
    t = torch.zeros(2, 2, dtype=torch.float16)
    with pytest.warns(UserWarning, match="C\\+\\+ module is not there"), pytest.raises(TypeError, match="x must be"):
        binding.lordba_forward(*[t] * 7)
    with pytest.raises(TypeError, match="x must be"):   # (said once)
        binding.lordba_forward(*[t] * 7)


@pytest.mark.gpu
def test_calls_without_the_module_give_the_same(monkeypatch):
    g = torch.Generator().manual_seed(6)
    half = lambda *s: torch.randn(s, generator=g).half().cuda()
    lat = torch.randn(8, 64, generator=g).cuda(), torch.randn(48, 8, generator=g).cuda()
    x, yb, s = half(5, 64), half(5, 48), (half(64), half(8), half(48))

    def calls():
        pA, pB, pAt, pBt = binding.lordba_pack_latents(*lat)
        y, t = binding.lordba_forward_save_t(x, pA, pB, *s, y_base=yb)
        d = binding.lordba_backward(x, yb, pA, pAt, pBt, *s, *lat, 100.0, dx_base=x.clone(), t_saved=t)
        return [binding.lordba_forward(x, pA, pB, *s, yb), y, pA, pB, pAt, pBt] + list(d.values())

    with_it = calls()
    _without_module(monkeypatch)
    with pytest.warns(UserWarning):
        without = calls()
    assert binding._torch_module is False
    assert all(torch.equal(a, b) for a, b in zip(with_it, without))
