"""The 64x128 and 128x128 tiles with two wavefront groups to a workgroup, which few tiles of sixteen stages and more run."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_19438_amd import workloads
from tests.test_gpu_scratch import COUNTERS, workspace

pytestmark = pytest.mark.gpu


# stages: 16 (the fewest), 17 (the groups' shares differ), 33 of which two slices get 17 and 16, a last half stage, a short last slice
@pytest.mark.parametrize("tile", [3, 5])
@pytest.mark.parametrize("M,K,N,group,split", [(65, 1024, 8, 128, 1), (128, 1088, 160, 64, 1), (129, 2112, 288, 64, 2), (200, 1056, 264, 32, 1),
                                               (100, 2080, 136, 32, 2), (257, 3200, 128, 128, 3), (70, 1120, 1032, 160, 1)])
def test_two_groups_match_the_oracle(tile, M, K, N, group, split):
    from paper_2511_19438_amd import binding as B

    case = workloads.make_case(M, K, N, group, seed=K + M)
    dev = {k: torch.from_numpy(case[k]).cuda() for k in ("x", "qweight", "qzeros", "scales")}
    out, again = (torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    for o in (out, again):
        B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, o, group, B.Plan(kernel=2, tile=tile, split_k=split))
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.maximum(1.0, np.abs(ref)))
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))


# automatic slices of both tiles, the plain variant and the one with a group row per half stage (small groups or a width of 8
# mod 32), sixteen to 26 stages to a slice, a last half stage and a short last slice
@pytest.mark.parametrize("tile", [3, 5])
@pytest.mark.parametrize("M,K,N,group", [(257, 8192, 544, 128), (129, 6144, 288, 64), (130, 8192, 1032, 128), (200, 8224, 264, 32), (300, 8192, 1024, 32)])
def test_two_groups_give_the_bits_of_the_form_without_scratch(tile, M, K, N, group):
    from paper_2511_19438_amd import binding as B

    plan = B.Plan(kernel=2, tile=tile)
    split = B.gptq_w4a16_plan_query(M, K, N, group, False, plan).split_k
    stages = -(-K // 64)
    per_slice = -(-stages // split)
    tiles = -(-M // (128 if tile == 3 else 64)) * -(-N // 128)
    assert split > 1 and per_slice >= 16 and -(-tiles // 8) * split <= 32, "two groups"
    case = workloads.make_case(M, K, N, group, seed=M)
    dev = {k: torch.from_numpy(case[k]).cuda() for k in ("x", "qweight", "qzeros", "scales")}
    sliced, walked = (torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, sliced, group, plan)
    with workspace(B, COUNTERS):
        B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, walked, group, plan)
        torch.cuda.synchronize()
    assert torch.equal(sliced.view(torch.int16), walked.view(torch.int16))
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    assert np.all(np.abs(sliced.cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.maximum(1.0, np.abs(ref)))


# other rows to a workgroup than the tile's own, where they pad less: 80, 96 and 112 rows of both widths, one group and two, whole
# and half stages, a last half stage, rows on both sides of a tile's edge, with and without scratch for the slices
@pytest.mark.parametrize("tile,M,K,N,group,split", [(5, 65, 1024, 136, 128, 1), (5, 80, 704, 1032, 64, 2), (5, 81, 1088, 288, 64, 1), (5, 96, 2112, 264, 32, 2),
                                                    (5, 97, 640, 520, 128, 1), (5, 112, 1056, 136, 32, 1), (5, 333, 2112, 128, 64, 2),
                                                    (8, 77, 1024, 264, 128, 1), (8, 80, 1120, 520, 32, 2), (8, 65, 512, 256, 128, 1),
                                                    (8, 112, 2112, 288, 64, 2), (8, 97, 1056, 40, 32, 1), (8, 222, 448, 544, 64, 1)])
def test_rows_that_fit_the_batch(tile, M, K, N, group, split):
    from paper_2511_19438_amd import binding as B

    case = workloads.make_case(M, K, N, group, seed=K + M)
    dev = {k: torch.from_numpy(case[k]).cuda() for k in ("x", "qweight", "qzeros", "scales")}
    plan = B.Plan(kernel=2, tile=tile, split_k=split)
    assert B.gptq_w4a16_plan_query(M, K, N, group, False, plan).split_k == split
    dev["x"][M - 1, K - 1] = float("inf")  # reaches its own row alone
    out, again = (torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    for o in (out, again):
        B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, o, group, plan)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)[:M - 1]
    assert np.all(np.abs(out[:M - 1].cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.maximum(1.0, np.abs(ref)))
    assert not np.isfinite(out[M - 1].float().cpu().numpy()).any()
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))


# the big-tile kernel in the mid-batch kernel's place, and plans that a query gave: the same bits, also without scratch
@pytest.mark.parametrize("M,K,N,group", [(100, 11008, 520, 128), (77, 8192, 8192, 128), (65, 9216, 704, 64), (64, 8192, 10240, 128)])
def test_in_the_mid_batch_kernels_place(M, K, N, group):
    from paper_2511_19438_amd import binding as B

    resolved = B.gptq_w4a16_plan_query(M, K, N, group)
    assert resolved.kernel == 4 and resolved.tile in (3, 5, 8) and resolved.split_k > 1
    case = workloads.make_case(M, K, N, group, seed=M)
    dev = {k: torch.from_numpy(case[k]).cuda() for k in ("x", "qweight", "qzeros", "scales")}
    auto, back, walked = (torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(3))
    B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, auto, group)
    B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, back, group, resolved)
    with workspace(B, COUNTERS):
        B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, walked, group)
        torch.cuda.synchronize()
    assert torch.equal(auto.view(torch.int16), back.view(torch.int16)) and torch.equal(auto.view(torch.int16), walked.view(torch.int16))
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    assert np.all(np.abs(auto.cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.maximum(1.0, np.abs(ref)))
