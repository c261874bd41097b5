"""What the binding does where the native code is not built."""
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
