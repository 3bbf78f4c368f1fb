"""build() needs hipcc alone for the library: without torch, a host compiler or Python's
headers it leaves the binding's native module out, and no earlier one behind."""
import os

import pytest

from paper_2606_26631_amd import build as b


@pytest.fixture
def steps(monkeypatch, tmp_path):
    """build() with its compiler runs replaced; returns what was linked."""
    linked = []
    monkeypatch.setattr(b, "BUILD_DIR", str(tmp_path))
    monkeypatch.setattr(b, "_compile", lambda src, verbose: src + ".o")
    monkeypatch.setattr(b, "_link", lambda objs, out, verbose: linked.append(out))
    monkeypatch.setattr(b, "_link_native", lambda obj, verbose: linked.append(b.NATIVE_OUT))
    monkeypatch.setattr(b, "NATIVE_OUT", str(tmp_path / "_prcr_native.so"))
    (tmp_path / "_prcr_native.so").write_text("an earlier build's")
    return linked


@pytest.mark.parametrize("missing", ["compiler", "torch", "headers"])
def test_library_is_built_without_the_native_module(steps, monkeypatch, tmp_path, capsys, missing):
    if missing == "compiler":
        monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    elif missing == "torch":
        monkeypatch.setitem(b.sys.modules, "torch.utils.cpp_extension", None)
    else:
        monkeypatch.setattr(b.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert b.build() == b.OUT
    assert steps == [b.OUT, b.COPYREF_OUT]
    assert not os.path.exists(b.NATIVE_OUT)
    assert "native module" in capsys.readouterr().err


def test_a_failing_compile_is_not_passed_over(steps, monkeypatch):
    def fails(verbose):
        raise RuntimeError("the host compiler failed")
    monkeypatch.setattr(b, "_compile_native", fails)
    with pytest.raises(RuntimeError, match="host compiler"):
        b.build()
    assert steps == [b.OUT, b.COPYREF_OUT] and not os.path.exists(b.NATIVE_OUT)
