"""The binding's extension module is an accelerator: everything but its speed is there without it (CPU)."""
import os

import pytest

torch = pytest.importorskip("torch")

from paper_2511_19438_amd import binding as B  # noqa: E402
from paper_2511_19438_amd import build  # noqa: E402


@pytest.fixture
def fresh(monkeypatch):
    """The binding as it is before load()."""
    if not os.path.exists(B.LIB_PATH):
        build.build()
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_native_gemm", None)
    return monkeypatch


def works_without_a_device():
    assert B.gptq_w4a16_plan_query(8, 4096, 4096, 128).kernel == 3
    assert B.gptq_w4a16_workspace_bytes(8, 4096, 4096, 128) > 0 and B.strerror(-3)
    x, qw, qz = torch.zeros(2, 128, dtype=torch.float16), torch.zeros(16, 8, dtype=torch.int32), torch.zeros(1, 1, dtype=torch.int32)
    sc, out, perm = torch.ones(1, 8, dtype=torch.float16), torch.zeros(2, 8, dtype=torch.float16), torch.arange(128, dtype=torch.int32)
    for call in (lambda: B.gptq_w4a16_gemm(x, qw, qz, sc, None, out, 128), lambda: B.gptq_w4a16_gemm_static(x, qw, qz, sc, None, out, 128),
                 lambda: B.gptq_w4a16_gemm_prepared(x, qw, qz, sc, perm, out, 128)):
        with pytest.raises(ValueError, match="device memory"):
            call()


def test_the_library_loads_with_and_without_the_module(fresh, tmp_path):
    B.load()
    if torch.version.hip and os.path.exists(build.native_call_path()):
        assert B._native_gemm is not None
    works_without_a_device()
    broken = tmp_path / "broken.so"
    broken.write_bytes(b"no shared object")
    for path in (tmp_path / "absent.so", broken):
        fresh.setattr(B, "_lib", None)
        fresh.setattr(B, "native_call_path", lambda: str(path))
        B.load()
        assert B._native_gemm is None
        works_without_a_device()


def test_a_module_of_another_torch_is_not_loaded(fresh):
    built = build.native_call_path()
    fresh.setattr(torch, "__version__", "0.0.0")
    assert build.native_call_path() != built and not os.path.exists(build.native_call_path())
    B.load()
    assert B._native_gemm is None


def test_the_build_goes_on_without_the_module(fresh, tmp_path):
    fresh.setattr(build, "LIB_DIR", str(tmp_path))
    for compiler in ("/bin/false", str(tmp_path / "no such compiler")):
        fresh.setenv("CXX", compiler)
        with pytest.warns(UserWarning, match="not built"):
            assert build.build_native_call() is None
    assert not list(tmp_path.iterdir())


def test_the_module_is_there_with_a_torch_that_has_gpu_support():
    if not torch.version.hip:
        pytest.skip("a torch without GPU support")
    if not os.path.exists(build.native_call_path()):
        assert build.build_native_call()
    assert B._load_native_call(build.native_call_path()) is not None
