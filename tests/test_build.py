"""The C library is built whether or not the binding's compiled calls can be (no torch, no g++, no Python headers)."""
import sys

import pytest

from paper_2509_23202_amd import build


@pytest.fixture
def linked(tmp_path, monkeypatch):
    """A build into tmp_path whose compiler writes an empty output file."""
    hipcc = tmp_path / "hipcc"
    hipcc.write_text('#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\n: > "$2"\n')
    hipcc.chmod(0o755)
    monkeypatch.setattr(build, "HIPCC", str(hipcc))
    monkeypatch.setattr(build, "BUILD", tmp_path / "objects")
    monkeypatch.setattr(build, "LIB", tmp_path / "libfp4mr.so")
    monkeypatch.setattr(build, "CALLS", tmp_path / "_calls.so")
    build.CALLS.write_text("of another build")

    def run():
        build.build(verbose=False)
        return build.LIB.exists(), build.CALLS.exists()

    return run


def test_without_torch(linked, monkeypatch, capfd):
    monkeypatch.setitem(sys.modules, "torch", None)   # (import torch raises ImportError)
    assert linked() == (True, False)
    assert "_calls.so" in capfd.readouterr().err


def test_without_a_host_compiler(linked, monkeypatch, capfd):
    pytest.importorskip("torch")
    monkeypatch.setenv("CXX", "/no/such/compiler")
    assert linked() == (True, False)
    assert "_calls.so" in capfd.readouterr().err


def test_a_compiler_error_of_the_library_is_raised(linked, monkeypatch):
    monkeypatch.setattr(build, "HIPCC", "/bin/false")
    with pytest.raises(RuntimeError, match="hipcc failed"):
        linked()
