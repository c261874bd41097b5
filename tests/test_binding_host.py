"""What the binding does where the native code is not built, or does not load."""
import os
import sys

import pytest

from paper_2503_06671_amd import binding


@pytest.fixture
def nothing_built(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "libesc_convattn.so"))
    monkeypatch.setattr(binding, "_native", binding._NativeModule())


def test_estimator_weights_need_no_library(nothing_built):
    gen = binding.GenParams(None)
    assert gen.tensors == (None,) * 4
    with pytest.raises(FileNotFoundError):
        gen.handle


def test_a_native_half_that_does_not_load_says_why(nothing_built, monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", object())   # the library itself is there
    monkeypatch.setattr(binding, "NATIVE_PATH", str(tmp_path / "_native.so"))
    with pytest.raises(FileNotFoundError, match="_native.so is not built"):
        binding.GenParams(None).handle
    (tmp_path / "_native.so").write_bytes(b"no shared object")
    monkeypatch.setattr(sys.modules["paper_2503_06671_amd"], "__path__", [str(tmp_path)])
    monkeypatch.delitem(sys.modules, "paper_2503_06671_amd._native", raising=False)
    assert os.path.exists(binding.NATIVE_PATH)
    with pytest.raises(ImportError, match="_native.so"):
        binding.GenParams(None).handle
