"""The build without what only the binding's optional module needs."""
import os

import pytest

from paper_2603_06731_amd import build


@pytest.mark.parametrize("compiler", ["/nonexistent/c++", "false"])
def test_marshalling_module_that_cannot_be_built(compiler, monkeypatch, tmp_path, capsys):
    """A missing or failing C++ compiler does not end the build, and leaves no module of earlier sources behind."""
    module = tmp_path / "_marshal.so"
    module.write_bytes(b"of earlier sources")
    monkeypatch.setattr(build, "MARSHAL", str(module))
    monkeypatch.setenv("CXX", compiler)
    build.build_marshal(force=True)
    assert "ctypes" in capsys.readouterr().out and os.listdir(tmp_path) == []


def test_marshalling_module_up_to_date(monkeypatch, tmp_path):
    module = tmp_path / "_marshal.so"
    module.write_bytes(b"")
    monkeypatch.setattr(build, "MARSHAL", str(module))
    monkeypatch.setenv("CXX", "/nonexistent/c++")
    build.build_marshal()                    # newer than its sources: not compiled
    assert module.exists()
