"""The binding's native marshalling: plain calls take it, everything else meets the Python code's answers (GPU)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_19438_amd import workloads  # noqa: E402
from test_gpu_parity import B, dev, run_gemm  # noqa: E402,F401

M, K, N, GROUP = 4, 256, 72, 128


def tensors(act=False):
    case = workloads.make_case(M, K, N, GROUP, seed=3, act_order=act)
    t = {k: (None if case[k] is None else dev(case[k])) for k in ("x", "qweight", "qzeros", "scales", "g_idx")}
    t["out"] = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    return t


def call(B, t, static=False):
    f = B.gptq_w4a16_gemm_static if static else B.gptq_w4a16_gemm
    return f(t["x"], t["qweight"], t["qzeros"], t["scales"], t["g_idx"], t["out"], GROUP)


class Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("act", [False, True])
def test_the_same_result_with_and_without(B, act, monkeypatch):
    t = tensors(act)
    assert call(B, t) is t["out"]
    native = t["out"].clone()
    call(B, t, static=True)
    assert torch.equal(t["out"], native)
    monkeypatch.setattr(B, "_native_gemm", lambda *a: None)
    t["out"].zero_()
    call(B, t)
    assert torch.equal(t["out"], native) and native.any()
    monkeypatch.undo()
    t["out"].zero_()
    t["x"] = t["x"].as_subclass(Sub)
    call(B, t)
    assert torch.equal(t["out"], native)


@pytest.mark.parametrize("name,change,error", [
    ("x", lambda v: v.float(), TypeError), ("x", lambda v: v.cpu(), ValueError), ("x", lambda v: v[:, ::2], ValueError),
    ("x", lambda v: torch.cat([v, v], 1)[:, :K], ValueError), ("qweight", lambda v: v.long(), TypeError),
    ("qweight", lambda v: v[0], ValueError), ("qzeros", lambda v: v[:1], ValueError), ("scales", lambda v: v.t(), ValueError),
    ("g_idx", lambda v: torch.zeros(K - 1, dtype=torch.int32, device="cuda"), ValueError),
    ("g_idx", lambda v: torch.zeros(K, dtype=torch.int64, device="cuda"), TypeError),
    ("out", lambda v: v[:2], ValueError), ("out", lambda v: torch.zeros((N, M), dtype=torch.float16, device="cuda").t(), ValueError),
    ("x", lambda v: None, AttributeError)])
def test_calls_that_are_not_plain(B, name, change, error):
    t = tensors()
    t[name] = change(t[name])
    with pytest.raises(error):
        call(B, t)


def test_status_codes_and_transforms(B):
    t = tensors()
    t["x"] = torch.zeros(M * K + 1, dtype=torch.float16, device="cuda")[1:].view(M, K)  # 2 bytes past a 16-byte boundary
    with pytest.raises(B.GptqError) as e:
        call(B, t)
    assert e.value.code == -3
    t = tensors()
    with pytest.raises(RuntimeError):
        torch.vmap(lambda x: B.gptq_w4a16_gemm(x, t["qweight"], t["qzeros"], t["scales"], None, t["out"], GROUP))(t["x"][None])
    with torch.cuda.stream(torch.cuda.Stream()):
        call(B, t)
    torch.cuda.synchronize()
    side = t["out"].clone()
    call(B, t)
    assert torch.equal(side, t["out"])
    with pytest.raises(B.GptqError):
        B.gptq_w4a16_gemm(t["x"], t["qweight"], t["qzeros"], t["scales"], None, t["out"], -GROUP)
