"""The small-batch kernel on its ring of LDS slots: edges of tiles, rows, shares and slices against the oracle (GPU)."""
import numpy as np
import pytest

import oracle
from paper_2511_19438_amd import workloads
from tests.test_gpu_parity import assert_within_band, run_gemm
from tests.test_gpu_scratch import COUNTERS, bits, vector_scratch, workspace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2511_19438_amd import binding

    binding.load()
    return binding


def check(B, M, K, N, group, plan):
    case = workloads.make_case(M, K, N, group, seed=M + K + N)
    got = run_gemm(B, case, group, plan)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    assert_within_band(got, ref, f"{M}x{K}x{N} group {group}")
    return case, got


# one unit of 128 k (seven idle wavefronts), shares of one and two units, a last share cut short, slices of uneven length;
# rows on both sides of every change of the loads; widths that end inside a tile, inside its first 32 columns, and short of it
@pytest.mark.parametrize("tile", [32, 64, 96, 128])
@pytest.mark.parametrize("M,K,N,group,split_k", [
    (2, 128, 8, 128, 1), (8, 1152, 136, 128, 1), (9, 2176, 264, 128, 2), (16, 1024, 200, 1024, 1), (17, 1280, 72, 256, 3),
    (24, 2304, 104, 128, 1), (25, 1152, 328, 384, 2), (32, 2048, 520, 128, 1),
    (5, 1152, 136, 64, 1), (16, 1280, 104, 32, 2), (24, 1152, 72, 64, 2), (32, 1024, 328, 32, 1)])
def test_edges(B, tile, M, K, N, group, split_k):
    plan = B.Plan(kernel=3, tile=tile, split_k=split_k)
    resolved = B.gptq_w4a16_plan_query(M, K, N, group, False, plan)
    assert (resolved.kernel, resolved.tile, resolved.split_k) == (3, tile, split_k)
    check(B, M, K, N, group, plan)


# three row blocks in every width that they have, four in 32 columns: rows on both sides of every change of the loads
@pytest.mark.parametrize("M,K,N,group,split_k,tiles", [
    (33, 128, 8, 128, 1, (32, 64, 96)), (40, 1152, 328, 384, 2, (32, 64, 96)), (41, 2176, 104, 128, 3, (32, 64, 96)),
    (48, 1280, 264, 128, 1, (32, 64, 96)), (49, 1152, 136, 128, 2, (32,)), (56, 1280, 72, 256, 1, (32,)), (57, 2176, 104, 128, 3, (32,)),
    (64, 1024, 328, 128, 1, (32,))])
def test_more_than_two_row_blocks(B, M, K, N, group, split_k, tiles):
    for tile in tiles:
        plan = B.Plan(kernel=3, tile=tile, split_k=split_k)
        resolved = B.gptq_w4a16_plan_query(M, K, N, group, False, plan)
        assert (resolved.kernel, resolved.tile, resolved.split_k) == (3, tile, split_k)
        check(B, M, K, N, group, plan)


# in the mid-batch kernel's place, with the slices in parallel or without scratch for them
@pytest.mark.parametrize("M,K,N,group,sliced", [(33, 4096, 1032, 64, True), (40, 11008, 520, 128, True), (48, 8192, 264, 64, True),
                                                (48, 640, 257 * 96 + 8, 128, False), (56, 5120, 520, 64, True), (64, 8192, 264, 128, True),
                                                (49, 640, 8192, 128, False)])
def test_up_to_64_rows_under_the_mid_batch_kernels_id(B, M, K, N, group, sliced):
    resolved = B.gptq_w4a16_plan_query(M, K, N, group)
    assert resolved.kernel == 4 and (resolved.split_k > 1) == sliced and resolved.tile <= (96 if M <= 48 else 32)
    case, got = check(B, M, K, N, group, None)
    assert np.array_equal(bits(run_gemm(B, case, group, resolved)), bits(got))
    with workspace(B, COUNTERS):
        assert np.array_equal(bits(run_gemm(B, case, group)), bits(got))


# more workgroups than compute units: four wavefronts each
@pytest.mark.parametrize("M,tile,group", [(3, 32, 128), (12, 32, 32), (20, 32, 128), (32, 32, 64), (8, 64, 128), (32, 64, 128)])
def test_four_wavefronts(B, M, tile, group):
    check(B, M, 640, 257 * tile + 8, group, B.Plan(kernel=3, tile=tile, split_k=1))


# the mid-batch kernel's id up to 32 rows, as automatic plans and explicit ones have it
@pytest.mark.parametrize("M,K,N,plan", [(17, 1024, 10248, None), (32, 1024, 10248, None), (24, 2048, 264, dict(kernel=4)),
                                        (24, 2048, 264, dict(kernel=4, tile=96, split_k=2)), (1, 2048, 264, dict(kernel=4))])
def test_under_the_mid_batch_kernels_id(B, M, K, N, plan):
    plan = B.Plan(**plan) if plan else None
    resolved = B.gptq_w4a16_plan_query(M, K, N, 128, False, plan)
    assert resolved.kernel == 4
    case, got = check(B, M, K, N, 128, plan)
    assert np.array_equal(bits(run_gemm(B, case, 128, resolved)), bits(got))
    same = B.Plan(kernel=3, tile=resolved.tile, split_k=resolved.split_k)
    assert np.array_equal(bits(run_gemm(B, case, 128, same)), bits(got))


@pytest.mark.parametrize("M,K,N,group", [(2, 11008, 512, 128), (8, 4096, 1000, 128), (16, 8192, 264, 32), (20, 11008, 1024, 128),
                                         (32, 8192, 520, 64)])
def test_the_result_does_not_depend_on_the_scratch(B, M, K, N, group):
    resolved = B.gptq_w4a16_plan_query(M, K, N, group)
    assert resolved.kernel == 3 and resolved.split_k > 1
    case = workloads.make_case(M, K, N, group, seed=M)
    sliced = run_gemm(B, case, group)
    with workspace(B, vector_scratch(B, M, K, N, group, False) if M <= 16 else COUNTERS):
        assert np.array_equal(bits(run_gemm(B, case, group)), bits(sliced))


@pytest.mark.parametrize("kernel,tile", [(4, 0), (4, 32), (4, 64), (4, 96), (4, 128), (3, 32), (3, 96)])
def test_nor_does_it_under_a_plan_that_leaves_the_slices_open(B, kernel, tile):
    """(In slices made for wider tiles this layer's 32- and 96-column ones would be more workgroups than compute units.)"""
    M, K, N, group = 24, 8192, 4096, 128
    plan = B.Plan(kernel=kernel, tile=tile)
    assert B.gptq_w4a16_plan_query(M, K, N, group, False, plan).split_k > 1
    case, sliced = check(B, M, K, N, group, plan)
    with workspace(B, COUNTERS):
        assert np.array_equal(bits(run_gemm(B, case, group, plan)), bits(sliced))


def test_rows_of_other_batches_do_not_matter(B):
    """Row blocks are padded with rows that repeat, and infinities stay in their own row."""
    case = workloads.make_case(32, 1024, 264, 128, seed=5)
    whole = run_gemm(B, case, 128, B.Plan(kernel=3, tile=32, split_k=1))
    for M in (1, 7, 8, 15, 16, 23, 24, 31):
        part = run_gemm(B, dict(case, x=np.ascontiguousarray(case["x"][:M])), 128, B.Plan(kernel=3, tile=32, split_k=1))
        assert np.array_equal(bits(part), bits(whole[:M])), M
    x = case["x"].copy()
    x[3, 5] = np.inf
    got = run_gemm(B, dict(case, x=x), 128, B.Plan(kernel=3, tile=32, split_k=1))
    keep = [m for m in range(32) if m != 3]
    assert np.array_equal(bits(got[keep]), bits(whole[keep])) and not np.isfinite(got[3]).any()


# on the library's scratch the two slices swap their sums pair by pair, on a caller's workspace they go through it
@pytest.mark.parametrize("M,K,N,tile,group", [(2, 1024, 136, 32, 128), (13, 1152, 264, 64, 32), (32, 2048, 520, 96, 128),
                                              (24, 4096, 40, 128, 64)])
def test_two_slices_both_ways(B, M, K, N, tile, group):
    plan = B.Plan(kernel=3, tile=tile, split_k=2)
    case, swapped = check(B, M, K, N, group, plan)
    for _ in range(3):  # (the slots are empty again)
        assert np.array_equal(bits(run_gemm(B, case, group, plan)), bits(swapped))
    with workspace(B, COUNTERS + 2 * M * N * 4):
        assert np.array_equal(bits(run_gemm(B, case, group, plan)), bits(swapped))
    x = case["x"].copy()
    x[0, :] = np.inf  # partial sums that are infinite and, their difference, not a number
    x[1, 3] = np.nan
    got = run_gemm(B, dict(case, x=x), group, plan)
    assert not np.isfinite(got[:2]).any() and np.array_equal(bits(got[2:]), bits(swapped[2:]))
    assert np.array_equal(bits(run_gemm(B, case, group, plan)), bits(swapped))
