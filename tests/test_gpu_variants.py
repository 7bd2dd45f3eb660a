"""GPU parity of the kernel variants that the automatic plan picks by size, group and alignment, at the sizes where a
tile, a slice or a pipeline step ends, against the CPU oracle.  Bars as in test_gpu_parity.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2511_19438_amd import workloads  # noqa: E402
from test_gpu_parity import B, assert_within_band, dev, run_gemm  # noqa: E402,F401


def check(B, case, group, what, plan=None):
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    out = run_gemm(B, case, group, plan)
    assert_within_band(out, ref, what)
    return out


# ---- act-order as stored: rows 2 ... several row tiles, one unit per slice, groups of every size, any map ----

@pytest.mark.parametrize("M", [2, 16, 17, 32, 33, 64, 65, 130])
@pytest.mark.parametrize("K,N,group", [(128, 8, 8), (1152, 72, 128), (2048, 200, 32), (1280, 1032, 640)])
def test_act_order_lookup_variant(B, M, K, N, group):
    case = workloads.make_case(M, K, N, group, seed=M + K + N, act_order=True)
    check(B, case, group, f"act-order {M}x{K}x{N} group {group}")
    # a map that is no permutation of whole groups: some groups own many rows, some none
    case["g_idx"] = (np.random.default_rng(M).integers(0, K // group, K) ** 2 // max(1, K // group)).astype(np.int32)
    first = check(B, case, group, f"unbalanced map {M}x{K}x{N} group {group}")
    assert np.array_equal(first.view(np.uint16), run_gemm(B, case, group).view(np.uint16))


@pytest.mark.parametrize("M", [8, 40])
def test_act_order_runs_on_a_workspace_without_room_for_slices(B, M):
    """Scratch that holds no partial sums: from 17 rows on the call gives up its slices, below it is refused as before."""
    K, N, group = 2048, 264, 128
    case = workloads.make_case(M, K, N, group, seed=M, act_order=True)
    assert B.gptq_w4a16_plan_query(M, K, N, group, True).split_k > 1
    buf = torch.empty(1 << 18, dtype=torch.uint8, device="cuda")  # the arrival counters alone
    B.gptq_w4a16_set_workspace(buf)
    try:
        if M <= 16:
            with pytest.raises(B.GptqError) as e:
                run_gemm(B, case, group)
            assert e.value.code == -5
        else:
            check(B, case, group, "without slices")
    finally:
        B.gptq_w4a16_set_workspace(None)
