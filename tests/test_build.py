"""What a build leaves behind when a part of it fails (host only; one small source is compiled)."""
import os

import pytest

from paper_2605_17447_amd import _build


@pytest.fixture
def paths(monkeypatch, tmp_path):
    monkeypatch.setattr(_build, "SOURCES", ["probe.hip"])
    monkeypatch.setattr(_build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(_build, "CALL_LIB", str(tmp_path / "call.so"))
    (tmp_path / "call.so").write_bytes(b"of older sources")
    return tmp_path


def _missing(*a):
    raise FileNotFoundError("no compiler")


@pytest.mark.parametrize("command", [lambda out, *a: ["sh", "-c", f"echo no Python.h; : > {out}; exit 1"], _missing])
def test_the_library_is_built_without_the_call_extension(monkeypatch, paths, capfd, command):
    monkeypatch.setattr(_build, "_call_command", command)
    assert _build.build() == _build.LIB and os.path.exists(_build.LIB)
    assert sorted(os.listdir(paths)) == ["lib.so"]                     # nor an extension of older sources, nor half of one
    assert "no Python.h" in (err := capfd.readouterr().err) or "no compiler" in err


def test_a_source_that_fails_leaves_what_was_there(monkeypatch, paths):
    (paths / "bad.hip").write_text("this is no code\n")
    monkeypatch.setattr(_build, "SOURCES", [str(paths / "bad.hip")])       # (an absolute path stays as it is)
    monkeypatch.setattr(_build, "_call_command", lambda out, *a: ["sh", "-c", f": > {out}"])
    with pytest.raises(RuntimeError):
        _build.build()
    assert sorted(os.listdir(paths)) == ["bad.hip", "call.so"] and (paths / "call.so").read_bytes() == b"of older sources"
