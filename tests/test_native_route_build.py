"""The native route of the tensor calls is optional: the C library is built and
the binding works where it cannot be built, does not load or is of another
build."""
import os
import subprocess
import sys
import types
import warnings

import pytest

from paper_1502_02389_amd import build, lift as B

NAME = "paper_1502_02389_amd._tensor_calls"


def test_library_links_without_the_route(tmp_path, monkeypatch, capsys):
    old = tmp_path / "_tensor_calls.so"
    old.write_bytes(b"of an earlier build")
    monkeypatch.setattr(build, "TENSOR_CALLS", str(old))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "liblift.so"))
    monkeypatch.setattr(build, "BUILD", str(tmp_path))
    monkeypatch.setattr(build, "write_tuned_table", lambda: 0)
    monkeypatch.setattr(build, "_compile", lambda src, sanitize=False: "x.o")

    def run(cmd, **kw):     # the C++ compiler is not there, the linker is
        if cmd[0] != build.HIPCC:
            raise FileNotFoundError(cmd[0])
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(build.subprocess, "run", run)
    assert build.build() == str(tmp_path / "liblift.so") and os.path.exists(build.LIB)
    assert not old.exists()
    assert "is not built" in capsys.readouterr().err


def _loaded():
    with warnings.catch_warnings(record=True) as w:
        warnings.simplefilter("always")
        return B._load_native(), [str(x.message) for x in w]


@pytest.mark.parametrize("module", [types.ModuleType(NAME), types.SimpleNamespace(INTERFACE=B._INTERFACE - 1)])
def test_another_build_is_left_out(monkeypatch, module):
    monkeypatch.setitem(sys.modules, NAME, module)
    native, said = _loaded()
    assert native is B._NoNative and len(said) == 1 and "interface" in said[0]


def test_the_same_build_is_taken(monkeypatch):
    module = types.SimpleNamespace(INTERFACE=B._INTERFACE)
    monkeypatch.setitem(sys.modules, NAME, module)
    assert _loaded() == (module, [])


def test_absent_and_broken(monkeypatch):
    import importlib

    def absent(name):
        raise ModuleNotFoundError(name, name=name)

    def broken(name):
        raise ImportError("undefined symbol")

    monkeypatch.setattr(importlib, "import_module", absent)
    assert _loaded() == (B._NoNative, [])
    monkeypatch.setattr(importlib, "import_module", broken)
    native, said = _loaded()
    assert native is B._NoNative and "undefined symbol" in said[0]
