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


def test_plain_calls_take_the_module(B, monkeypatch):
    native = B._native_gemm
    assert native is not None
    codes = []
    monkeypatch.setattr(B, "_native_gemm", lambda *a: codes.append(native(*a)) or codes[-1])
    t = tensors()
    call(B, t)
    call(B, t, static=True)
    call(B, dict(t, x=t["x"].as_subclass(Sub)))
    assert codes == [0, 0, None]


@pytest.mark.parametrize("static", [False, True])
def test_the_module_enqueues_on_the_current_stream(B, static):
    """What the call reads is there late in its stream, and only for a while."""
    t = tensors()
    call(B, t, static)
    torch.cuda.synchronize()
    want, x = t["out"].clone(), t["x"].clone()
    big = torch.randn(4096, 4096, device="cuda")
    side = torch.cuda.Stream()
    t["x"].zero_()
    t["out"].zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(20):
            torch.mm(big, big)  # tens of milliseconds ahead of the copy
        t["x"].copy_(x)
        call(B, t, static)
        t["x"].zero_()
    torch.cuda.synchronize()
    assert torch.equal(t["out"], want)  # (on the default stream it would have read zeros)
    graph = torch.cuda.CUDAGraph()
    t["x"].copy_(x)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        call(B, t, static)
    for _ in range(3):
        t["out"].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(t["out"], want)  # (on another stream it would not be in the graph)
