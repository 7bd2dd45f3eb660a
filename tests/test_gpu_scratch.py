"""What a call does where the scratch of its K slices cannot be had (GPU): a caller's workspace that is too small, growth
while the stream is captured, the static block.  Bars as in test_gpu_parity.py."""
import contextlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2511_19438_amd import workloads  # noqa: E402
from test_gpu_parity import B, assert_within_band, dev, run_gemm  # noqa: E402,F401

COUNTERS = 1 << 18  # the arrival counters alone


@contextlib.contextmanager
def workspace(B, nbytes):
    B.gptq_w4a16_set_workspace(torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
    try:
        yield
    finally:
        B.gptq_w4a16_set_workspace(None)


def bits(a):
    return a.view(np.uint16)


@pytest.mark.parametrize("M,group,act,plan", [
    (40, 32, False, dict(kernel=2, tile=8, split_k=3)), (40, 32, False, dict(kernel=2, split_k=3)),
    (40, 32, False, dict(split_k=3)), (40, 128, True, dict(split_k=2)), (40, 128, True, dict(kernel=2, split_k=2, flags=16)),
    (8, 128, True, dict(kernel=1, split_k=2, flags=16)), (24, 32, False, dict(kernel=3, split_k=2))])
def test_an_explicit_number_of_slices_is_refused_without_their_scratch(B, M, group, act, plan):
    K, N = 2048, 264
    case = workloads.make_case(M, K, N, group, seed=M, act_order=act)
    plan = B.Plan(**plan)
    assert B.gptq_w4a16_plan_query(M, K, N, group, act, plan).split_k > 1
    with workspace(B, COUNTERS):
        with pytest.raises(B.GptqError) as e:
            run_gemm(B, case, group, plan)
        assert e.value.code == -5
