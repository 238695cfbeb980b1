"""The package without the native half of its binding, or with one that does not load: the C library is what it needs."""
import os
import warnings

import pytest

import paper_2605_08587_amd as kla

pytestmark = pytest.mark.skipif(not os.path.exists(kla.LIB_PATH), reason="libkla.so not built")


@pytest.mark.parametrize("form", ["missing", "garbage", "no module", "other PyTorch"])
def test_loads_without(monkeypatch, tmp_path, form):
    path = tmp_path / "kla_binding.so"
    if form == "garbage":
        path.write_bytes(b"not a library")
    if form == "other PyTorch":
        if not os.path.exists(kla.BINDING_PATH):
            pytest.skip("kla_binding.so not built")
        monkeypatch.setattr(kla.torch, "__version__", "1.0.0")
    else:
        monkeypatch.setattr(kla, "BINDING_PATH", kla.LIB_PATH if form == "no module" else str(path))
    monkeypatch.setattr(kla, "_lib", None)
    monkeypatch.setattr(kla, "_native", None)
    with warnings.catch_warnings(record=True) as seen:
        warnings.simplefilter("always")
        assert kla.kla_chunk_fwd_workspace_bytes(1, 64, 8, 128, 128, kla.torch.float32) > 0
    assert [w.category for w in seen] == ([] if form == "missing" else [RuntimeWarning])
    q = kla.torch.zeros(1, 1, 64)
    assert kla._binding().decode(q) is None and kla._binding().chunk_fwd(q) is None and kla._binding().chunk_bwd(q) is None
    with pytest.raises(RuntimeError, match="GPU tensors"):       # the step-by-step half takes the call, and refuses this one
        kla.kla_decode_step(q, q, q, q[..., 0], q[..., 0], 1e-6, kla.torch.zeros(1, 1, 64, 64))


def test_loads_with():
    if not os.path.exists(kla.BINDING_PATH):
        pytest.skip("kla_binding.so not built")
    assert kla._binding().__name__ == "kla_binding"
