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


# Rows to a workgroup other than the tile's own, where they pad less (the first seven: the tile's own, which the estimate keeps on
# narrow layers): tile, M, K, N, group, slices (0: as the plan has it), then the rows and the wavefront groups that the plan has for
# it.  80, 96 and 112 rows of both widths, one group and two, whole and half stages - a check on the CPU holds the list to that -,
# a last half stage, one row tile and several, rows on both sides of a tile's edge.
ROWS_THAT_FIT = [
    (5, 65, 1024, 136, 128, 1, 64, 2), (5, 80, 704, 1032, 64, 2, 64, 1), (5, 81, 1088, 288, 64, 1, 64, 2),
    (5, 96, 2112, 264, 32, 2, 64, 2), (5, 97, 640, 520, 128, 1, 64, 1), (5, 112, 1056, 136, 32, 1, 64, 2),
    (5, 333, 2112, 128, 64, 2, 64, 2), (8, 77, 1024, 264, 128, 1, 80, 2), (8, 80, 1120, 520, 32, 2, 80, 2),
    (8, 65, 512, 256, 128, 1, 80, 1), (8, 112, 2112, 288, 64, 2, 112, 2), (8, 97, 1056, 40, 32, 1, 112, 2),
    (8, 222, 448, 544, 64, 1, 80, 1), (5, 65, 2112, 8416, 64, 0, 80, 1), (5, 80, 3392, 5216, 64, 0, 80, 2),
    (5, 66, 1696, 5136, 32, 0, 80, 1), (5, 79, 2912, 5216, 32, 0, 80, 2), (5, 160, 384, 10912, 128, 0, 80, 1),
    (5, 129, 320, 10968, 160, 0, 80, 1), (5, 80, 1024, 17152, 64, 0, 80, 2), (5, 81, 2432, 8288, 64, 0, 96, 1),
    (5, 96, 3904, 5152, 64, 0, 96, 2), (5, 95, 1728, 5936, 96, 0, 96, 1), (5, 96, 2016, 8480, 96, 0, 96, 2),
    (5, 192, 1024, 11032, 32, 0, 96, 2), (5, 161, 384, 11424, 128, 0, 96, 1), (5, 333, 2752, 6888, 32, 0, 96, 2),
    (5, 82, 992, 16424, 32, 0, 96, 2), (5, 97, 2496, 8640, 64, 0, 112, 1), (5, 112, 2944, 8384, 128, 0, 112, 2),
    (5, 111, 2080, 8504, 160, 0, 112, 1), (5, 97, 2912, 8464, 32, 0, 112, 2), (5, 66, 384, 16576, 128, 0, 112, 1),
    (5, 65, 320, 16568, 160, 0, 112, 1), (5, 224, 1024, 8224, 64, 0, 80, 2), (8, 65, 1152, 32, 64, 0, 80, 1),
    (8, 80, 1920, 32, 128, 0, 80, 2), (8, 79, 960, 40, 160, 0, 80, 1), (8, 65, 2240, 40, 160, 0, 80, 2),
    (8, 160, 576, 320, 64, 0, 80, 2), (8, 96, 1152, 32, 128, 2, 96, 2), (8, 96, 448, 32, 64, 0, 96, 1),
    (8, 90, 1408, 32, 128, 0, 96, 2), (8, 95, 1344, 56, 96, 0, 96, 1), (8, 81, 1248, 56, 32, 0, 96, 2),
    (8, 192, 1344, 264, 96, 0, 80, 1), (8, 190, 384, 32, 128, 3, 80, 1), (8, 97, 1344, 256, 64, 0, 112, 1),
    (8, 112, 1536, 32, 64, 0, 112, 2), (8, 100, 1312, 264, 32, 0, 112, 1), (8, 111, 1280, 40, 32, 0, 112, 2),
    (8, 224, 512, 264, 128, 0, 80, 1),
]


@pytest.mark.parametrize("tile,M,K,N,group,split,rows,groups", ROWS_THAT_FIT)
def test_rows_that_fit_the_batch(tile, M, K, N, group, split, rows, groups):
    from paper_2511_19438_amd import binding as B

    case = workloads.make_case(M, K, N, group, seed=K + M)
    dev = {k: torch.from_numpy(case[k]).cuda() for k in ("x", "qweight", "qzeros", "scales")}
    plan = B.Plan(kernel=2, tile=tile, split_k=split)
    slices = B.gptq_w4a16_plan_query(M, K, N, group, False, plan).split_k
    assert split in (0, slices)
    dev["x"][M - 1, K - 1] = float("inf")  # reaches its own row alone
    out, again = (torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    for o in (out, again):
        B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, o, group, plan)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)[:M - 1]
    assert np.all(np.abs(out[:M - 1].cpu().numpy().astype(np.float64) - ref) <= 2e-2 * np.maximum(1.0, np.abs(ref)))
    assert not np.isfinite(out[M - 1].float().cpu().numpy()).any()
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))
    if split == 0 and slices > 1:  # the same without scratch for the slices
        with workspace(B, COUNTERS):
            B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, again, group, plan)
            torch.cuda.synchronize()
        finite = out[:M - 1].view(torch.int16), again[:M - 1].view(torch.int16)
        assert torch.equal(*finite) and not np.isfinite(again[M - 1].float().cpu().numpy()).any()


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
