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
@pytest.mark.parametrize("K,N,group", [(128, 8, 8), (1152, 72, 128), (2048, 200, 32), (1280, 1032, 640),
                                       (32, 8, 32), (1120, 136, 32), (2144, 72, 8), (1088, 264, 64)])  # K ends inside a unit
def test_act_order_lookup_variant(B, M, K, N, group):
    case = workloads.make_case(M, K, N, group, seed=M + K + N, act_order=True)
    check(B, case, group, f"act-order {M}x{K}x{N} group {group}")
    # a map that is no permutation of whole groups: some groups own many rows, some none
    case["g_idx"] = (np.random.default_rng(M).integers(0, K // group, K) ** 2 // max(1, K // group)).astype(np.int32)
    first = check(B, case, group, f"unbalanced map {M}x{K}x{N} group {group}")
    assert np.array_equal(first.view(np.uint16), run_gemm(B, case, group).view(np.uint16))


@pytest.mark.parametrize("M,K,group", [(2, 28672, 64), (17, 19392, 32), (40, 19392, 32)])  # 448 and 606 groups
def test_act_order_lookup_variant_with_tables_as_large_as_the_lds(B, M, K, group):
    case = workloads.make_case(M, K, 72, group, seed=M, act_order=True)
    assert B.gptq_w4a16_plan_query(M, K, 72, group, True).tile == 64
    check(B, case, group, f"{K // group} groups, M={M}")


@pytest.mark.parametrize("M,K,N,group", [(2, 1280, 264, 128), (8, 4096, 1032, 128), (16, 1376, 4104, 32), (40, 2048, 264, 64),
                                         (130, 4096, 520, 128)])
def test_a_queried_act_order_plan_runs_the_automatic_call_again(B, M, K, N, group):
    case = workloads.make_case(M, K, N, group, seed=M, act_order=True)
    plan = B.gptq_w4a16_plan_query(M, K, N, group, True)
    assert plan.flags == 16
    assert np.array_equal(run_gemm(B, case, group, plan).view(np.uint16), run_gemm(B, case, group).view(np.uint16))
    check(B, case, group, "three slices", B.Plan(kernel=plan.kernel, split_k=3, flags=16))


@pytest.mark.parametrize("M", [8, 40])
def test_act_order_runs_on_a_workspace_without_room_for_slices(B, M):
    """Scratch that holds no partial sums: from 17 rows on the workgroups walk the slices themselves, below the call is refused."""
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


@pytest.mark.parametrize("M", [2, 8, 16, 17, 32])
@pytest.mark.parametrize("K,N,group,split_k", [(32, 8, 32, 1), (96, 72, 32, 1), (160, 264, 32, 2), (192, 136, 64, 1),
                                               (1120, 520, 32, 3), (1984, 1032, 64, 4), (4128, 4104, 32, 0)])
def test_small_batch_kernel_with_a_k_that_ends_inside_a_unit(B, M, K, N, group, split_k):
    case = workloads.make_case(M, K, N, group, seed=M + K + N)
    plan = B.Plan(kernel=3 if split_k else 0, split_k=split_k)
    assert B.gptq_w4a16_plan_query(M, K, N, group, False, plan).kernel == (3 if split_k or M > 2 else 1)
    check(B, case, group, f"small batch {M}x{K}x{N} group {group} split {split_k}", plan)
    if not split_k and M <= 2:
        return  # the vector kernel: biased codes, an infinity leaves it as a NaN
    # an infinity in the last 32 k, which the steps past K load again, must reach its own row only, and not as a NaN
    case["x"][0, K - 3] = np.float16(np.inf)
    out = run_gemm(B, case, group, plan).astype(np.float64)
    w = oracle.dequant(case["qweight"], case["qzeros"], case["scales"], None, group)[K - 3].astype(np.float64)
    assert np.array_equal(np.isnan(out[0]), w == 0) and np.all(np.isfinite(out[1:]))


# ---- big-tile kernel with a row of scales and zero points per 32-k half stage: groups that are odd multiples of 32, a K
#      that ends half-way through a stage, widths that are no multiple of 32; every tile, with and without K slices ----

@pytest.mark.parametrize("tile", [1, 3, 5, 8])
@pytest.mark.parametrize("M,K,N,group,split_k", [
    (70, 64, 8, 32, 1),        # one stage
    (130, 96, 40, 32, 1),      # K ends in the second stage, three groups of one half each
    (65, 96, 264, 96, 2),      # a slice that is nothing but the half-repeated last stage
    (257, 160, 520, 32, 1),    # ... in the third (cleared inside the loop)
    (33, 672, 136, 96, 3),     # groups of three halves, slices that start inside a group
    (300, 1056, 1032, 32, 4),
    (96, 512, 264, 128, 2),    # groups of whole stages, width no multiple of 32
])
def test_big_tile_half_stage_groups(B, tile, M, K, N, group, split_k):
    case = workloads.make_case(M, K, N, group, seed=M + K + N)
    plan = B.Plan(kernel=2, tile=tile, split_k=split_k)
    res = B.gptq_w4a16_plan_query(M, K, N, group, False, plan)
    assert res.kernel == 2 and res.tile == tile
    first = check(B, case, group, f"tile {tile} {M}x{K}x{N} group {group} split {split_k}", plan)
    assert np.array_equal(first.view(np.uint16), run_gemm(B, case, group, plan).view(np.uint16))


# ---- 128x256 tile: 80 and 96 rows where they fit the batch better, two wavefront groups per workgroup that halve its K slice ----

@pytest.mark.parametrize("M", [70, 96, 128, 130, 192])  # 80 rows; 96; 128; two tiles of 80; three
@pytest.mark.parametrize("K,N,group,split_k", [
    (512, 264, 128, 1),    # eight stages: one group
    (576, 264, 64, 1),     # nine: five and four
    (1280, 520, 128, 2),   # two slices of ten stages
    (608, 136, 32, 1),     # ends half-way through a stage, in the second group
    (1888, 40, 32, 3),     # slices of ten, ten and ten stages (the last one ends half-way)
    (1184, 72, 32, 2),     # slices of ten and nine stages: five and four, the last one half
])
def test_tile_of_two_wavefront_groups(B, M, K, N, group, split_k):
    case = workloads.make_case(M, K, N, group, seed=M + K + N)
    plan = B.Plan(kernel=2, tile=8, split_k=split_k)
    first = check(B, case, group, f"128x256 tile {M}x{K}x{N} group {group} split {split_k}", plan)
    assert np.array_equal(first.view(np.uint16), run_gemm(B, case, group, plan).view(np.uint16))


def test_half_stage_groups_repeat_nothing_of_a_row(B):
    """The last 64 k of a K that ends half-way through a stage contain 32 that the stage before has multiplied already:
    infinities among those activations must count once, like every other value."""
    M, K, N, group = 40, 160, 64, 32
    case = workloads.make_case(M, K, N, group, seed=3)
    case["x"][5, 100] = np.float16(np.inf)  # k 96 ... 127 are read twice
    out = run_gemm(B, case, group).astype(np.float64)
    w = oracle.dequant(case["qweight"], case["qzeros"], case["scales"], None, group)[100].astype(np.float64)
    assert np.array_equal(np.isnan(out[5]), w == 0) and np.all(out[5][w != 0] == np.sign(w[w != 0]) * np.inf)
    case["x"][5, 100] = np.float16(0)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    rows = np.arange(M) != 5
    assert_within_band(out[rows].astype(np.float16), ref[rows], "the other rows")


def test_half_stage_groups_run_on_a_workspace_without_room_for_slices(B):
    M, K, N, group = 40, 2048, 264, 32
    case = workloads.make_case(M, K, N, group, seed=M)
    assert B.gptq_w4a16_plan_query(M, K, N, group).split_k > 1
    B.gptq_w4a16_set_workspace(torch.empty(1 << 18, dtype=torch.uint8, device="cuda"))  # the arrival counters alone
    try:
        check(B, case, group, "without slices")
    finally:
        B.gptq_w4a16_set_workspace(None)


# ---- an infinity among the activations: its row is infinite where the weight is not zero, whatever the number of slices
#      (a slice count that the batches of the exchange do not divide must not turn it into a NaN) ----

@pytest.mark.parametrize("kernel,tile,M,group,split_k", [
    (2, 5, 70, 128, 3), (2, 5, 70, 32, 5), (2, 3, 70, 128, 3), (2, 3, 130, 32, 3), (2, 8, 130, 32, 3),
    (4, 64, 40, 128, 3), (4, 64, 90, 64, 3), (3, 64, 24, 32, 3), (0, 0, 40, 32, 0)])
def test_an_infinity_survives_the_exchange_of_k_slices(B, kernel, tile, M, group, split_k):
    K, N = 1536, 136  # (24 stages: every wavefront of the mid-batch kernel has whole stages of its own)
    case = workloads.make_case(M, K, N, group, seed=M + split_k)
    plan = B.Plan(kernel=kernel, tile=tile, split_k=split_k)
    resolved = B.gptq_w4a16_plan_query(M, K, N, group, False, plan)
    assert resolved.split_k > 1 and kernel in (0, resolved.kernel)
    w = oracle.dequant(case["qweight"], case["qzeros"], case["scales"], None, group).astype(np.float64)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    for k in (5, K - 7):  # in the first slice and in the last
        x = case["x"].copy()
        x[3, k] = np.float16(np.inf)
        out = run_gemm(B, dict(case, x=x), group, plan)
        assert np.array_equal(np.isnan(out[3]), w[k] == 0), f"infinity at k = {k}"
        hit = w[k] != 0
        assert np.array_equal(out[3][hit], (np.sign(w[k][hit]) * np.inf).astype(np.float16))
        rows = np.arange(M) != 3
        assert_within_band(out[rows], ref[rows], "the other rows")


@pytest.mark.parametrize("M,K,tile,split_k", [(40, 1280, 64, 3), (24, 1280, 128, 1), (64, 704, 64, 1), (90, 1344, 64, 2), (48, 2048, 0, 0)])
def test_an_infinity_counts_once_where_wavefronts_have_uneven_shares(B, M, K, tile, split_k):
    """Mid-batch kernel, and the ring in its place (40 and 24 rows): a wavefront with fewer stages than the others goes through
    its last bodies without a stage."""
    N, group = 136, 64
    case = workloads.make_case(M, K, N, group, seed=M)
    plan = B.Plan(kernel=4, tile=tile, split_k=split_k)
    resolved = B.gptq_w4a16_plan_query(M, K, N, group, False, plan)
    slices = [K // 64 // resolved.split_k * i for i in range(resolved.split_k + 1)]
    w = oracle.dequant(case["qweight"], case["qzeros"], case["scales"], None, group).astype(np.float64)
    for k in sorted({K - 1, K - 64, 64 * slices[1] - 3, 5}):
        x = case["x"].copy()
        x[M - 1, k] = np.float16(-np.inf)
        out = run_gemm(B, dict(case, x=x), group, plan)
        assert np.array_equal(np.isnan(out[M - 1]), w[k] == 0), f"k = {k}"
        assert np.all(np.isfinite(out[:M - 1]))


# ---- dequantisation: write-through stores up to 224 MB of output, past the caches beyond, plain ones at ragged widths ----

@pytest.mark.parametrize("act,group", [(False, 128), (True, 64)])
@pytest.mark.parametrize("K,N", [(8192, 13664), (8192, 13696), (8192, 13688), (1024, 32), (1024, 24)])  # 223.9 and 224.4 MB
def test_dequant_store_policies_are_bit_exact(B, K, N, group, act):
    w = workloads.make_weights(K, N, group, seed=K + N, act_order=act)
    qw, qz, sc, gi = (dev(w[k]) for k in ("qweight", "qzeros", "scales", "g_idx"))
    guard = torch.full((K + 2, N), 7.0, dtype=torch.float16, device="cuda")  # a row on either side stays as it is
    B.gptq_w4a16_dequant(qw, qz, sc, gi, guard[1:-1], group)
    shift = torch.arange(0, 32, 4, dtype=torch.int32, device="cuda")
    z = (qz[:, :, None] >> shift & 15).reshape(K // group, N)
    group_of = gi.long() if act else torch.arange(K, device="cuda") // group
    for lo in range(0, K, 1024):
        q = (qw[lo // 8:lo // 8 + 128, None, :] >> shift[None, :, None] & 15).reshape(1024, N)
        rows = group_of[lo:lo + 1024]
        want = (q - z[rows]).half() * sc[rows]  # exact difference, one fp16 multiplication
        assert torch.equal(guard[1 + lo:1 + lo + 1024].view(torch.int16), want.view(torch.int16)), lo
    assert bool((guard[0] == 7).all()) and bool((guard[-1] == 7).all())


@pytest.mark.parametrize("M", [2, 17, 130, 384])
def test_act_order_lookups_with_four_units_per_slice(B, M):
    K, N, group = 20160, 72, 32  # 630 groups: 40 slices
    case = workloads.make_case(M, K, N, group, seed=M, act_order=True)
    plan = B.gptq_w4a16_plan_query(M, K, N, group, True)
    assert (plan.flags, plan.split_k) == (16, 40)
    check(B, case, group, f"630 groups, M={M}")


# ---- non-temporal weight loads (matrices of 128 MB and more, rows of whole cache lines): every tile of both kernels ----

@pytest.fixture(scope="module", params=[(8192, 31264), (16384, 16384)], ids=str)  # 64-column tiles: four wavefronts, eight
def large(request, B):
    K, N, group = *request.param, 128
    assert N % 32 == 0 and K * N // 2 >= 128000000
    case = workloads.make_case(16, K, N, group, seed=N)
    qw, qz, sc, x = (dev(case[k]) for k in ("qweight", "qzeros", "scales", "x"))
    w = torch.empty((K, N), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_dequant(qw, qz, sc, None, w, group)  # bit-exact by its own tests
    ref = torch.cat([x.float() @ w[:, lo:lo + 4096].float() for lo in range(0, N, 4096)], dim=1).cpu().numpy()
    return x, qw, qz, sc, ref, group


@pytest.mark.parametrize("kernel,tile,split_k,batches", [
    (1, 64, 1, (1,)), (1, 64, 3, (1,)), (1, 128, 1, (1,)), (1, 128, 5, (1,)), (1, 256, 1, (1,)), (1, 256, 7, (1,)),
    (3, 64, 1, (2, 16)), (3, 64, 3, (2, 16)), (3, 128, 1, (2, 16)), (3, 128, 3, (2, 16)), (3, 256, 1, (2, 16)),
    (3, 256, 8, (2, 16)), (0, 0, 0, (1, 2, 7, 16))])
def test_streamed_weights(B, large, kernel, tile, split_k, batches):
    x, qw, qz, sc, ref, group = large
    for M in batches:
        out = torch.full((M, qw.shape[1]), float("nan"), dtype=torch.float16, device="cuda")
        B.gptq_w4a16_gemm(x[:M], qw, qz, sc, None, out, group, B.Plan(kernel=kernel, tile=tile, split_k=split_k))
        assert_within_band(out.cpu().numpy(), ref[:M], f"kernel {kernel} tile {tile} slices {split_k} M={M}")
