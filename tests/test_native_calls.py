"""The native calls are a faster way to the same library: without them, or with those of another torch,
the binding makes its own checks, and the build does without torch.  No GPU."""
import sys
import types

import pytest
import torch

from paper_2203_05016_amd import binding, build as lib_build, synth


@pytest.fixture(params=["missing", "another torch", "not a module"])
def no_native_calls(request, monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_calls", None)
    if request.param == "another torch":
        monkeypatch.setattr(torch, "__version__", "0.0.0")
    else:
        path = tmp_path / "_torch_calls.so"
        if request.param == "not a module":
            path.write_bytes(b"\x7fELF")
        monkeypatch.setattr(binding, "CALLS_PATH", str(path))


@pytest.mark.filterwarnings("ignore:native calls not in use")
def test_binding_works_without_native_calls(no_native_calls, monkeypatch):
    x = torch.zeros((16, 64), dtype=torch.float16)
    with pytest.raises(ValueError, match="one GPU"):   # the binding's own check
        binding.layernorm_transpose(x, out=torch.zeros((64, 16), dtype=torch.float16))
    assert binding.calls() is False
    p = synth.make_spmm(64, 40, 24, 32, 0.5, seed=7)
    A = binding.compress(p.W, p.mask, p.perm, p.V)
    A.info()
    monkeypatch.setattr(binding, "lib", lambda: types.SimpleNamespace(
        shflbw_bind_device=lambda *a: 0, shflbw_device_bytes=lambda h: 256))   # no GPU to copy to
    A.bind_device("cpu", stream=types.SimpleNamespace(cuda_stream=0))
    assert A._plan is None
    with pytest.raises(ValueError, match="K = 40"):
        A.spmm(x, torch.zeros((64, 64), dtype=torch.float16))


def test_missing_native_calls_are_reported_once(no_native_calls):
    with pytest.warns(UserWarning, match="native calls not in use"):
        binding.calls()
    import warnings
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert binding.calls() is False


def test_build_does_not_need_torch(monkeypatch):
    assert lib_build._torch_calls_command("out.so")[0] == "g++"
    with monkeypatch.context() as m:
        m.setitem(sys.modules, "torch", None)
        assert lib_build._torch_calls_command("out.so") is None
    from torch.utils import cpp_extension
    monkeypatch.setattr(cpp_extension, "include_paths", lambda *a, **k: [])
    assert lib_build._torch_calls_command("out.so") is None
