"""The Python entry points without their native module: one that is missing, or was built for
another torch or Python, costs speed and a warning, never a call."""
import sys
import types

import pytest
import torch

import paper_2606_26631_amd as prcr
from paper_2606_26631_amd import binding

NAME = "paper_2606_26631_amd._prcr_native"


def _without(monkeypatch, module):
    monkeypatch.setattr(binding, "_NATIVE", None)
    monkeypatch.delattr(prcr, "_prcr_native", raising=False)
    monkeypatch.setitem(sys.modules, NAME, module)


def _refused():
    """A call that the Python path refuses for its own reason (tensors of the CPU)."""
    cpu = torch.zeros(1, 2, 1, 1, 64)
    mem = types.SimpleNamespace(k=cpu, v=cpu, device=cpu.device)
    with pytest.raises(ValueError, match="raw_k must be a GPU tensor"):
        prcr.store_raw(mem, 0, cpu[0], cpu[0], torch.zeros(1, 2, dtype=torch.int32))


def test_a_missing_module_is_not_needed(monkeypatch):
    _without(monkeypatch, None)                 # import raises ImportError
    with pytest.warns(RuntimeWarning, match="native"):
        _refused()
    _refused()                                  # and is not looked for again


def test_a_module_of_another_torch_is_not_used(monkeypatch):
    other = types.ModuleType(NAME)
    other.built_for = "torch 0.1, Python 2.7"
    _without(monkeypatch, other)
    with pytest.warns(RuntimeWarning, match="torch 0.1"):
        _refused()


def test_the_module_built_here_is_used(monkeypatch, recwarn):
    monkeypatch.setattr(binding, "_NATIVE", None)
    assert binding._native().__name__ == NAME
    assert not [w for w in recwarn if issubclass(w.category, RuntimeWarning)]


def test_arguments_are_checked_before_the_library_is_loaded(monkeypatch, tmp_path):
    _without(monkeypatch, None)
    monkeypatch.setattr(binding, "_LIB", None)
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "libprcr.so"))
    with pytest.warns(RuntimeWarning):
        _refused()
