"""CPU-only: the library is built whether or not the C++ autograd nodes can be, and neither that nor their absence goes unsaid."""
import os

import pytest

from paper_2409_15373_amd import autograd, build


def test_the_library_is_built_without_the_nodes(monkeypatch, tmp_path, capsys):
    build.build()
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libjfa.so"))
    monkeypatch.setattr(build, "native_path", lambda version: str(tmp_path / "_native.so"))
    monkeypatch.setenv("CXX", "false")
    (tmp_path / "_native.so").write_bytes(b"of an older source")
    os.utime(tmp_path / "_native.so", (0, 0))
    assert os.path.exists(build.build()) and not os.path.exists(tmp_path / "_native.so")
    assert "autograd nodes are not built" in capsys.readouterr().err


@pytest.mark.parametrize("content", [None, b"not a library"])
def test_nodes_that_cannot_be_loaded(monkeypatch, tmp_path, content):
    path = tmp_path / "_native.so"
    if content:
        path.write_bytes(content)
    monkeypatch.setattr(autograd, "native_path", lambda version: str(path))
    monkeypatch.setattr(autograd, "_native", None)
    with pytest.warns(UserWarning, match="autograd nodes"):
        autograd._load_native()
    assert autograd._native is False


def test_another_torch_has_nodes_of_its_own():
    assert build.native_path("1.0") != build.native_path("2.0")
