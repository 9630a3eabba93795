"""What happens where the extension module _call.so is not there, not for this torch, or older than its source (no GPU needed):
the calls that it shortens go through ctypes, as they did without it, and the warnings name the file that they are about."""
import os
import sys
import warnings

import pytest
import torch

import paper_2411_00850_amd as gwq
from paper_2411_00850_amd import binding, build


@pytest.fixture
def not_bound(monkeypatch):
    monkeypatch.setattr(binding, "_plain_call", None)
    return monkeypatch


def _goes_through_ctypes():
    """One warning, and then the binding's own checks word the error."""
    with pytest.warns(UserWarning, match="_call.so is not used"):
        assert binding._plain()(None, None, None, False) is None
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        for fn in (gwq.linear, gwq.linear_bf16):
            with pytest.raises(AssertionError):
                fn(None, torch.zeros(1, 128))


def test_module_missing(not_bound):
    not_bound.setitem(sys.modules, "paper_2411_00850_amd._call", None)
    not_bound.delattr(gwq, "_call", raising=False)
    _goes_through_ctypes()


def test_module_of_another_torch(not_bound):
    not_bound.setattr(build, "built_for", lambda: "torch 1.0, Python 3.10")
    _goes_through_ctypes()


def test_library_builds_without_a_compiler_for_the_module(monkeypatch, tmp_path):
    call = tmp_path / "_call.so"
    call.write_text("of an earlier build")
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libgwq.so"))
    monkeypatch.setattr(build, "CALL", str(call))
    monkeypatch.setenv("HIPCC", "true")
    for compiler in ("false", str(tmp_path / "no-such-compiler")):
        monkeypatch.setenv("CXX", compiler)
        with pytest.warns(UserWarning, match="_call.so is not built"):
            assert build.build() == str(tmp_path / "libgwq.so")
        assert not call.exists()


def test_stale_names_the_file(monkeypatch, tmp_path):
    for name in ("libgwq.so", "_call.so", "gwq_call.cpp", "gwq_api.hip", "gwq_internal.h", "gwq.h"):
        (tmp_path / name).write_text("")
        os.utime(tmp_path / name, (1000, 1000))
    for name, value in (("LIB", "libgwq.so"), ("CALL", "_call.so"), ("CSRC", ""), ("INCLUDE", "")):
        monkeypatch.setattr(build, name, str(tmp_path / value))
    assert not build.stale()
    for source, built in (("gwq_call.cpp", ["_call.so"]), ("gwq_internal.h", ["libgwq.so"]), ("gwq.h", ["libgwq.so", "_call.so"])):
        os.utime(tmp_path / source, (2000, 2000))
        assert build.stale() == built
        os.utime(tmp_path / source, (1000, 1000))
    (tmp_path / "_call.so").unlink()
    assert not build.stale()
