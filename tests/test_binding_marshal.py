"""The binding without its marshalling module: calls go through ctypes, and a build that cannot make the module still makes the library."""
import warnings

import pytest
import torch

from paper_2411_04965_amd import binding as B
from paper_2411_04965_amd import build


def _load(monkeypatch, path):
    monkeypatch.setattr(B, "_marshal", None)
    monkeypatch.setattr(B, "MARSHAL_PATH", str(path))
    return B._native()


def test_absent_module(monkeypatch, tmp_path):
    """No module, or a file that cannot be loaded: ctypes, and one warning that says so."""
    (tmp_path / "broken.so").write_bytes(b"not a shared object")
    for name in ("absent.so", "broken.so"):
        with pytest.warns(RuntimeWarning, match="ctypes"):
            assert _load(monkeypatch, tmp_path / name) is False
        with warnings.catch_warnings():
            warnings.simplefilter("error")
            assert B._native() is False


def test_build_without_module(monkeypatch, tmp_path, capsys):
    """No C++ compiler: the library is built all the same, an older module goes."""
    old = tmp_path / "bitlinear_marshal.old.so"
    old.write_bytes(b"")
    monkeypatch.setattr(build, "LIB_DIR", str(tmp_path))
    monkeypatch.setattr(build, "_build_library", lambda verbose, jobs: None, raising=False)
    monkeypatch.setenv("CXX", str(tmp_path / "no-compiler"))
    assert build.build(verbose=False) == build.LIB
    assert not old.exists() and "ctypes" in capsys.readouterr().err


def test_one_module_for_each_torch(monkeypatch):
    """A module that was built with another torch is not taken."""
    assert B.MARSHAL_PATH == B._marshal_path()
    monkeypatch.setattr(torch, "__version__", "9.9.9")
    assert B._marshal_path() != B.MARSHAL_PATH
