"""The build of the library does not depend on the optional Python module."""
import importlib.machinery
import os

import pytest

from paper_2510_06175_amd import build


@pytest.mark.parametrize("command", [["/nonexistent/g++"], ["false"], None], ids=["no-compiler", "failing-compiler", "no-headers"])
def test_library_is_linked_without_the_native_module(command, tmp_path, monkeypatch, capfd):
    """(Every compile of the library is `true` here.)"""
    old = tmp_path / "_fastcall.so"
    old.write_bytes(b"of an earlier build")
    monkeypatch.setenv("HIPCC", "true")
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libvecinfer.so"))
    monkeypatch.setattr(build, "FASTCALL", str(old))
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "fastcall_command", lambda: command)
    assert build.build() == str(tmp_path / "libvecinfer.so")
    assert not os.path.exists(old)
    assert "calls go through ctypes" in capfd.readouterr().err


def test_the_native_module_is_this_interpreters_alone():
    """Another Python would load a plain `_fastcall.so`, though its internals may differ."""
    name = os.path.basename(build.FASTCALL)
    assert name == "_fastcall" + importlib.machinery.EXTENSION_SUFFIXES[0] and name != "_fastcall.so"
