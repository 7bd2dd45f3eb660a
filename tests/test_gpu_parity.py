"""GPU parity: the HIP library (through its C ABI) against the CPU oracle, element by element.

Bars: unpack and dequant bit-exact; GEMM within 2e-2 * max(1, |ref|) of the fp64-accumulated
reference on every element (and far inside it: fp32 accumulation should sit near one fp16 ulp).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2511_19438_amd import workloads  # noqa: E402

TOL = 2e-2


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_19438_amd import binding

    binding.load()  # raises if the HIP library is not built: there is no fallback to test
    return binding


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def run_gemm(B, case, group, plan=None):
    x, qw, qz, sc, gi = (dev(case[k]) for k in ("x", "qweight", "qzeros", "scales", "g_idx"))
    out = torch.full((x.shape[0], qw.shape[1]), float("nan"), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_gemm(x, qw, qz, sc, gi, out, group, plan)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def assert_within_band(out, ref, what, tight=0.25):
    out64 = out.astype(np.float64)
    assert np.all(np.isfinite(out64)), f"{what}: non-finite output"
    ratio = np.abs(out64 - ref) / (TOL * np.maximum(1.0, np.abs(ref)))
    worst = float(ratio.max())
    assert worst <= 1.0, f"{what}: max err/tol = {worst:.3f} at {np.unravel_index(ratio.argmax(), ratio.shape)}"
    # fp32 accumulation + one fp16 rounding: a correct kernel uses a small part of the band
    assert worst <= tight, f"{what}: err/tol = {worst:.3f} is suspiciously large for fp32 accumulation"
    return worst


# ------------------------------------------------------------------ unpack / dequant (bit-exact)

@pytest.mark.parametrize("K,N,group", [(128, 8, 128), (256, 72, 32), (1024, 1000, 128), (4096, 4096, 128), (384, 264, 64)])
def test_unpack_bit_exact(B, K, N, group):
    w = workloads.make_weights(K, N, group, seed=K + N)
    q_out = torch.empty((K, N), dtype=torch.uint8, device="cuda")
    z_out = torch.empty((K // group, N), dtype=torch.uint8, device="cuda")
    B.gptq_w4a16_unpack(dev(w["qweight"]), q_out, dev(w["qzeros"]), z_out, group)
    torch.cuda.synchronize()
    assert np.array_equal(q_out.cpu().numpy(), oracle.unpack_qweight(w["qweight"]))
    assert np.array_equal(z_out.cpu().numpy(), oracle.unpack_qzeros(w["qzeros"]))
    # z_out is optional
    q2 = torch.empty_like(q_out)
    B.gptq_w4a16_unpack(dev(w["qweight"]), q2, None, None, group)
    assert torch.equal(q2, q_out)


def test_unpack_hand_packed_words(B):
    qweight = np.array([[0x76543210, 0xF0000001, 0x8000000F, 0x11111111, 0, 0xFFFFFFFF, 0x0F0F0F0F, 0x12345678]],
                       np.uint32).view(np.int32)
    qzeros = np.array([[0xFEDCBA98]], np.uint32).view(np.int32)
    q_out = torch.empty((8, 8), dtype=torch.uint8, device="cuda")
    z_out = torch.empty((1, 8), dtype=torch.uint8, device="cuda")
    B.gptq_w4a16_unpack(dev(qweight), q_out, dev(qzeros), z_out, 8)
    q = q_out.cpu().numpy()
    assert q[:, 0].tolist() == [0, 1, 2, 3, 4, 5, 6, 7]
    assert q[:, 1].tolist() == [1, 0, 0, 0, 0, 0, 0, 15]
    assert q[:, 2].tolist() == [15, 0, 0, 0, 0, 0, 0, 8]
    assert q[:, 7].tolist() == [8, 7, 6, 5, 4, 3, 2, 1]
    assert z_out.cpu().numpy()[0].tolist() == [8, 9, 10, 11, 12, 13, 14, 15]


@pytest.mark.parametrize("K,N,group,act", [(128, 8, 128, False), (256, 72, 32, True), (1024, 1000, 128, False),
                                           (4096, 4096, 128, False), (4096, 11008, 128, True), (384, 264, 8, False),
                                           (512, 136, 512, True)])
def test_dequant_bit_exact(B, K, N, group, act):
    w = workloads.make_weights(K, N, group, seed=K + N + 1, act_order=act)
    w_out = torch.empty((K, N), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_dequant(dev(w["qweight"]), dev(w["qzeros"]), dev(w["scales"]), dev(w["g_idx"]), w_out, group)
    torch.cuda.synchronize()
    expected = oracle.dequant(w["qweight"], w["qzeros"], w["scales"], w["g_idx"], group)
    assert np.array_equal(w_out.cpu().numpy().view(np.uint16), expected.view(np.uint16))


def test_dequant_subnormal_negative_and_overflowing_scales(B):
    K, N, group = 64, 16, 32
    w = workloads.make_weights(K, N, group, seed=3)
    special = np.array([2.0 ** -24, 2.0 ** -20, 3 * 2.0 ** -24, -0.007, 30000.0, -30000.0, 6.1e-5, 1.0], np.float16)
    w["scales"] = np.tile(special, (K // group, N // 8)).astype(np.float16)
    w_out = torch.empty((K, N), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_dequant(dev(w["qweight"]), dev(w["qzeros"]), dev(w["scales"]), None, w_out, group)
    expected = oracle.dequant(w["qweight"], w["qzeros"], w["scales"], None, group)
    assert np.array_equal(w_out.cpu().numpy().view(np.uint16), expected.view(np.uint16))


def test_golden_dequant_samples(B):
    import os

    rows = [l.split() for l in open(os.path.join(os.path.dirname(__file__), "golden", "config0_dequant_samples.txt"))
            if not l.startswith("#")]
    w = workloads.make_weights(4096, 4096, 128, seed=workloads.case_seed(0))
    w_out = torch.empty((4096, 4096), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_dequant(dev(w["qweight"]), dev(w["qzeros"]), dev(w["scales"]), None, w_out, 128)
    got = w_out.cpu().numpy().view(np.uint16)
    for k, n, bits in rows:
        assert int(got[int(k), int(n)]) == int(bits, 16)


# ------------------------------------------------------------------ GEMM, vector (decode) kernel

DECODE_SHAPES = [
    # (K, N, group, act_order): several column tiles with a ragged last one, several K slices
    (1024, 200, 128, False),
    (2048, 1032, 128, False),
    (1024, 328, 128, True),
    (768, 136, 64, False),
    (512, 72, 32, True),
    (256, 64, 16, False),   # two packed rows per group: chunk of 2
    (192, 40, 24, False),   # three packed rows per group: chunk of 1
    (128, 8, 128, False),   # the smallest legal problem
]


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 8, 13, 16])
@pytest.mark.parametrize("K,N,group,act", DECODE_SHAPES)
def test_decode_gemm_matches_oracle(B, M, K, N, group, act):
    case = workloads.make_case(M, K, N, group, seed=10 * K + N + M, act_order=act)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    out = run_gemm(B, case, group)
    assert_within_band(out, ref, f"decode M={M} K={K} N={N} g={group} act={act}")


@pytest.mark.parametrize("tile", [16, 32, 64, 128, 256])
@pytest.mark.parametrize("split_k", [1, 2, 3, 7, 64])
@pytest.mark.parametrize("M", [1, 4, 16])
def test_decode_plans_match_oracle(B, tile, split_k, M):
    K, N, group = 2048, 776, 128
    case = workloads.make_case(M, K, N, group, seed=77 + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=1, split_k=split_k, tile=tile))
    assert_within_band(out, ref, f"plan tile={tile} split={split_k} M={M}")


@pytest.mark.parametrize("M,K,split_k", [(1, 11008, 1), (2, 11008, 1), (1, 16384, 1), (1, 16416, 1), (2, 16384, 3)])
def test_decode_deep_slices(B, M, K, split_k):
    """One workgroup walks the whole K (or the longest slice the LDS budget allows): many pipeline steps,
    a ragged last step, the activations of the slice filling the staging buffer."""
    N, group = 264, 32
    case = workloads.make_case(M, K, N, group, seed=K + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    for tile in (32, 128):
        out = run_gemm(B, case, group, B.Plan(kernel=1, split_k=split_k, tile=tile))
        assert_within_band(out, ref, f"deep slice M={M} K={K} tile={tile}")


@pytest.mark.parametrize("flags", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("M,split_k", [(1, 0), (1, 3), (2, 0), (3, 1), (4, 2)])
def test_ablation_variants_match_oracle(B, flags, M, split_k):
    """Each of the paper's three techniques taken out in turn (and together): the baselines they replace
    compute the same result, inside the same band (the atomic commit adds in no fixed order)."""
    K, N, group = 2048, 776, 128
    case = workloads.make_case(M, K, N, group, seed=900 + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    for _ in range(2):  # twice: the arrival counters must be back at zero, the sums zeroed again
        out = run_gemm(B, case, group, B.Plan(kernel=1, split_k=split_k, flags=flags))
        assert_within_band(out, ref, f"ablation flags={flags} M={M} split={split_k}")


def test_vector_kernel_handles_batches_above_16(B):
    M, K, N, group = 37, 512, 136, 128
    case = workloads.make_case(M, K, N, group, seed=5)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=1))
    assert_within_band(out, ref, "vector kernel M=37")


# ------------------------------------------------------------------ GEMM, MFMA (prefill) kernel

PREFILL_CASES = [
    # (M, K, N, group, act_order)
    (17, 256, 72, 128, False),
    (64, 512, 256, 128, False),
    (100, 1024, 328, 128, False),
    (256, 512, 512, 64, False),
    (300, 768, 264, 128, False),
    (513, 1024, 520, 128, False),
    (96, 256, 136, 32, False),    # group per packed row mode
    (40, 216, 72, 24, False),     # K not a multiple of the 64-wide stage
    (130, 512, 200, 128, True),   # act-order mode
    (33, 264, 40, 8, True),
]


@pytest.mark.parametrize("M,K,N,group,act", PREFILL_CASES)
def test_prefill_gemm_matches_oracle(B, M, K, N, group, act):
    case = workloads.make_case(M, K, N, group, seed=M + K + N, act_order=act)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    out = run_gemm(B, case, group)
    assert_within_band(out, ref, f"prefill M={M} K={K} N={N} g={group} act={act}")


@pytest.mark.parametrize("tile", [1, 3, 5, 8])
@pytest.mark.parametrize("M,N", [(300, 328), (32, 520), (300, 544), (1, 256)])
def test_prefill_tiles_match_oracle(B, tile, M, N):
    K, group = 1024, 128
    case = workloads.make_case(M, K, N, group, seed=tile + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=2, tile=tile))
    assert_within_band(out, ref, f"prefill tile={tile} M={M} N={N}")


@pytest.mark.parametrize("tile", [1, 3, 5, 8])
@pytest.mark.parametrize("split_k", [2, 3, 7, 32])
@pytest.mark.parametrize("M,N", [(300, 544), (40, 288)])
def test_prefill_k_split_matches_oracle(B, tile, split_k, M, N):
    """K slices of the big-tile kernel (slices that end inside a group, a ragged last slice, more slices
    requested than stages), combined through scratch; twice in a row: the arrival counters must be back at zero."""
    K, group = 1408, 128   # 22 stages of 64 k
    case = workloads.make_case(M, K, N, group, seed=tile + M + split_k)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    plan = B.Plan(kernel=2, tile=tile, split_k=split_k)
    res = B.gptq_w4a16_plan_query(M, K, N, group, False, plan)
    assert res.kernel == 2 and res.tile == tile and res.split_k >= 2
    first = run_gemm(B, case, group, plan)
    again = run_gemm(B, case, group, plan)
    assert_within_band(first, ref, f"prefill tile={tile} split={split_k} M={M} N={N}")
    assert np.array_equal(first.view(np.uint16), again.view(np.uint16))


def test_mfma_kernel_also_serves_small_batches_when_asked(B):
    M, K, N, group = 3, 512, 264, 128
    case = workloads.make_case(M, K, N, group, seed=8)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=2))
    assert_within_band(out, ref, "mfma M=3")


# ------------------------------------------------------------------ GEMM, small-batch MFMA kernel

SKINNY_SHAPES = [
    # (K, N, group): several column tiles with a ragged last one, several K slices, units not a multiple of 4
    (1024, 200, 128),
    (2048, 1032, 128),
    (640, 72, 128),
    (1536, 328, 256),
    (128, 8, 128),
]


@pytest.mark.parametrize("tile", [64, 128, 256])
@pytest.mark.parametrize("M", [1, 5, 8, 16, 17, 32, 33, 49, 64, 65, 100, 128])
@pytest.mark.parametrize("K,N,group", SKINNY_SHAPES)
def test_small_batch_mfma_kernel_matches_oracle(B, M, K, N, group, tile):
    case = workloads.make_case(M, K, N, group, seed=3 * K + N + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=3, tile=tile))
    assert_within_band(out, ref, f"small-batch M={M} K={K} N={N} g={group} tile={tile}")


@pytest.mark.parametrize("tile", [64, 128, 256])
@pytest.mark.parametrize("split_k", [1, 2, 3, 5, 16])
@pytest.mark.parametrize("M", [8, 40, 64, 90])
def test_small_batch_mfma_kernel_splits(B, split_k, M, tile):
    K, N, group = 2048, 776, 128
    case = workloads.make_case(M, K, N, group, seed=177 + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=3, split_k=split_k, tile=tile))
    assert_within_band(out, ref, f"small-batch split={split_k} M={M} tile={tile}")


@pytest.mark.parametrize("group", [64, 32])
@pytest.mark.parametrize("M", [2, 8, 16, 17, 32])
@pytest.mark.parametrize("K,N,split_k", [(1024, 200, 0), (2048, 1032, 3), (640, 72, 0), (128, 8, 0)])
def test_small_batch_mfma_kernel_small_groups(B, M, K, N, split_k, group):
    """Groups of 64 and 32 k: two / four (scale, zero) rows per 128-k unit, the MFMA chain scaled per group."""
    assert B.gptq_w4a16_plan_query(M, K, N, group).kernel == 3, "the small-batch kernel is the default here"
    case = workloads.make_case(M, K, N, group, seed=5 * K + N + M + group)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=3, split_k=split_k))
    assert_within_band(out, ref, f"small-batch M={M} K={K} N={N} g={group}")


@pytest.mark.parametrize("group", [64, 32])
def test_small_batch_small_groups_one_hot_rows_bit_exact(B, group):
    M, K, N = 12, 1024, 264
    w = workloads.make_weights(K, N, group, seed=19 + group)
    hot = [(131 * m + 7) % K for m in range(M)]
    case = dict(w, x=workloads.one_hot_activations(M, K, hot))
    w16 = oracle.dequant(w["qweight"], w["qzeros"], w["scales"], None, group)
    out = run_gemm(B, case, group, B.Plan(kernel=3))
    for m, j in enumerate(hot):
        assert np.array_equal(out[m].view(np.uint16), w16[j].view(np.uint16)), f"row {m} (k={j})"


def test_small_batch_request_falls_back_when_unsupported(B):
    # act-order and group sizes that are not multiples of 128 are served by the other kernels
    for M, K, N, group, act in [(8, 512, 136, 16, False), (8, 192, 136, 64, False), (40, 512, 136, 64, False),
                                (8, 512, 136, 128, True), (200, 512, 136, 128, False)]:
        case = workloads.make_case(M, K, N, group, seed=M + N, act_order=act)
        ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
        out = run_gemm(B, case, group, B.Plan(kernel=3))
        assert_within_band(out, ref, f"fallback M={M} g={group} act={act}")


# ------------------------------------------------------------------ GEMM, mid-batch streaming MFMA kernel
# (up to 32 rows, and in 64 columns up to 48, the ring runs in its place where K is a multiple of 128)

MID_SHAPES = [
    # (K, N, group): several column tiles with a ragged last one; stage counts that are not multiples of three or of
    # the wavefront count (a single stage included); groups of one, two, three and four 64-k stages
    (1024, 200, 128),
    (2048, 1032, 128),
    (640, 72, 64),
    (1536, 328, 256),
    (64, 8, 64),
    (1152, 136, 192),
]


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("M", [1, 17, 32, 33, 49, 64, 65, 100, 128])
@pytest.mark.parametrize("K,N,group", MID_SHAPES)
def test_mid_batch_kernel_matches_oracle(B, M, K, N, group, tile):
    case = workloads.make_case(M, K, N, group, seed=3 * K + N + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    plan = B.Plan(kernel=4, tile=tile)
    res = B.gptq_w4a16_plan_query(M, K, N, group, False, plan)
    assert res.kernel == 4 and res.tile == (tile if M <= 64 else 64)  # four row blocks: 64-column tiles only
    out = run_gemm(B, case, group, plan)
    assert_within_band(out, ref, f"mid-batch M={M} K={K} N={N} g={group} tile={tile}")


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("split_k", [1, 2, 3, 5, 32])
@pytest.mark.parametrize("M", [40, 64, 90])
def test_mid_batch_kernel_splits(B, split_k, M, tile):
    """K slices across workgroups (ragged last slice, more slices than a wavefront has stages), combined through
    scratch; twice in a row: the arrival counters must be back at zero and the result the same bit for bit."""
    K, N, group = 2048, 776, 128
    case = workloads.make_case(M, K, N, group, seed=177 + M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    plan = B.Plan(kernel=4, split_k=split_k, tile=tile)
    first = run_gemm(B, case, group, plan)
    again = run_gemm(B, case, group, plan)
    assert_within_band(first, ref, f"mid-batch split={split_k} M={M} tile={tile}")
    assert np.array_equal(first.view(np.uint16), again.view(np.uint16))


def test_mid_batch_request_falls_back_when_unsupported(B):
    # act-order, K or group sizes that are not multiples of 64, more than 128 rows: served by the other kernels
    for M, K, N, group, act in [(40, 512, 136, 32, False), (40, 160, 136, 32, False), (40, 512, 136, 128, True),
                                (200, 512, 136, 128, False)]:
        assert B.gptq_w4a16_plan_query(M, K, N, group, act, B.Plan(kernel=4)).kernel != 4
        case = workloads.make_case(M, K, N, group, seed=M + N, act_order=act)
        ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
        out = run_gemm(B, case, group, B.Plan(kernel=4))
        assert_within_band(out, ref, f"fallback M={M} g={group} act={act}")


# ------------------------------------------------------------------ exactness pins in the GEMM kernels themselves

@pytest.mark.parametrize("M,plan_kernel", [(1, 1), (4, 1), (8, 1), (16, 1), (40, 2), (300, 2), (8, 3), (24, 3), (40, 3), (64, 3),
                                           (20, 4), (48, 4), (100, 4)])
@pytest.mark.parametrize("act", [False, True])
def test_one_hot_rows_return_weight_rows_bit_exact(B, M, plan_kernel, act):
    K, N, group = 1024, 264, 128
    w = workloads.make_weights(K, N, group, seed=9, act_order=act)
    hot = [(131 * m + 7) % K for m in range(M)]
    case = dict(w, x=workloads.one_hot_activations(M, K, hot))
    w16 = oracle.dequant(w["qweight"], w["qzeros"], w["scales"], w["g_idx"], group)
    out = run_gemm(B, case, group, B.Plan(kernel=plan_kernel))
    for m, j in enumerate(hot):
        assert np.array_equal(out[m].view(np.uint16), w16[j].view(np.uint16)), f"row {m} (k={j})"


@pytest.mark.parametrize("M", [1, 8, 64, 100, 200])
def test_dyadic_scales_and_ternary_activations_are_exact(B, M):
    # scales 2^-7, x in {-1,0,1}: every partial sum is an exact dyadic rational, so fp32 accumulation in any
    # order equals the fp64 reference and the fp16 result is its single rounding
    K, N, group = 1024, 328, 128
    case = workloads.make_weights(K, N, group, seed=12)
    case["scales"] = np.full_like(case["scales"], 2.0 ** -7)
    case["x"] = workloads.ternary_activations(M, K, seed=M)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    out = run_gemm(B, case, group)
    assert np.array_equal(out.view(np.uint16), oracle.double_to_half_bits(ref))


@pytest.mark.parametrize("M", [1, 2, 8, 48, 80])
def test_codes_equal_to_zero_points_give_zero(B, M):
    K, N, group = 512, 136, 128
    z = np.random.default_rng(4).integers(0, 16, size=(K // group, N), dtype=np.uint8)
    case = {"qweight": oracle.pack_qweight(np.repeat(z, group, axis=0)), "qzeros": oracle.pack_qzeros(z),
            "scales": np.full((K // group, N), 0.01, np.float16), "g_idx": None,
            "x": workloads.make_activations(M, K, seed=4)}
    out = run_gemm(B, case, group)
    if M > 1:
        # exact q - z before the contraction (all three MFMA kernels): every product is exactly zero
        assert np.all(out == 0)
    else:
        # the single-row vector kernel contracts the biased codes (1024 + q) and takes the bias and the zero
        # point off per 32-k chunk in fp32: the cancellation leaves fp32 rounding noise of the order
        # 1e-3 * scale, far inside the tolerance band around a reference of exactly zero
        assert np.all(np.abs(out.astype(np.float64)) <= 1e-3)


def test_trivial_g_idx_equals_null_and_calls_are_deterministic(B):
    M, K, N, group = 4, 1024, 264, 128
    case = workloads.make_case(M, K, N, group, seed=21)
    a = run_gemm(B, case, group)
    b = run_gemm(B, case, group)
    assert np.array_equal(a.view(np.uint16), b.view(np.uint16))
    case_g = dict(case, g_idx=(np.arange(K) // group).astype(np.int32))
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    assert_within_band(run_gemm(B, case_g, group), ref, "explicit trivial g_idx")


def test_caller_owned_workspace(B):
    M, K, N, group = 8, 2048, 520, 128
    case = workloads.make_case(M, K, N, group, seed=33)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    need = B.gptq_w4a16_workspace_bytes(M, K, N, group)
    assert need > 0
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    B.gptq_w4a16_set_workspace(ws)
    try:
        assert_within_band(run_gemm(B, case, group), ref, "caller workspace")
        with pytest.raises(B.GptqError) as err:  # no room for the arrival counters
            B.gptq_w4a16_set_workspace(torch.empty(4096, dtype=torch.uint8, device="cuda"))
        assert err.value.code == -5
        small = torch.empty(300 * 1024, dtype=torch.uint8, device="cuda")  # counters fit, the partial sums do not
        B.gptq_w4a16_set_workspace(small)
        with pytest.raises(B.GptqError) as err:
            run_gemm(B, case, group, B.Plan(kernel=1, split_k=8))
        assert err.value.code == -5
    finally:
        B.gptq_w4a16_set_workspace(None)
    assert_within_band(run_gemm(B, case, group), ref, "library workspace again")


def test_golden_gemm_samples_config0(B):
    import os

    rows = [l.split() for l in open(os.path.join(os.path.dirname(__file__), "golden", "config0_gemm_samples.txt"))
            if not l.startswith("#")]
    case = workloads.make_case(1, 4096, 4096, 128, seed=workloads.case_seed(0))
    out = run_gemm(B, case, 128)
    for m, n, v in rows:
        ref = float.fromhex(v)
        assert abs(float(out[int(m), int(n)]) - ref) <= TOL * max(1.0, abs(ref))


def test_scratch_survives_a_change_of_problem_width(B):
    # Regression: the arrival counters of the split-K combine sit at a fixed place in the scratch.  A wide
    # problem after a narrower one (whose partial sums once overlapped the wider one's counters) must still
    # write every output column.
    group = 128
    for N in (512, 4096, 1024, 12288, 2048):
        case = workloads.make_case(1, 1024, N, group, seed=N)
        ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
        out = run_gemm(B, case, group, B.Plan(kernel=1, split_k=4, tile=16))
        assert_within_band(out, ref, f"N={N} after other widths")


# ------------------------------------------------------------------ act-order repack (one-time) and its GEMM

REPACK_SHAPES = [(1024, 328, 128), (512, 72, 32), (2048, 1032, 128), (256, 64, 64)]


def _repack(B, case, group):
    qw = dev(case["qweight"])
    qs = torch.empty_like(qw)
    perm = torch.empty(case["g_idx"].shape[0], dtype=torch.int32, device="cuda")
    B.gptq_w4a16_act_order_prepare(qw, dev(case["g_idx"]), qs, perm, group)
    return qs, perm


@pytest.mark.parametrize("K,N,group", REPACK_SHAPES)
def test_repack_sorts_rows_by_group_bit_exact(B, K, N, group):
    """perm is the stable order of k by g_idx; the sorted matrix dequantises, without g_idx, to the rows of the
    oracle's act-order weights in that order."""
    case = workloads.make_case(1, K, N, group, seed=K + N, act_order=True)
    qs, perm = _repack(B, case, group)
    want_perm = np.argsort(case["g_idx"], kind="stable").astype(np.int32)
    assert np.array_equal(perm.cpu().numpy(), want_perm)
    w_ref = oracle.dequant(case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    w_out = torch.empty((K, N), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_dequant(qs, dev(case["qzeros"]), dev(case["scales"]), None, w_out, group)
    got = w_out.cpu().numpy().view(np.uint16)
    assert np.array_equal(got, w_ref.view(np.uint16)[want_perm])
    # and the codes themselves
    q_ref = oracle.unpack_qweight(case["qweight"])
    q_out = torch.empty((K, N), dtype=torch.uint8, device="cuda")
    B.gptq_w4a16_unpack(qs, q_out, None, None, group)
    assert np.array_equal(q_out.cpu().numpy(), q_ref[want_perm])


@pytest.mark.parametrize("M", [1, 2, 8, 16, 40, 300])
@pytest.mark.parametrize("K,N,group", REPACK_SHAPES[:3])
def test_repacked_gemm_matches_oracle(B, M, K, N, group):
    case = workloads.make_case(M, K, N, group, seed=7 * K + N + M, act_order=True)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    qs, perm = _repack(B, case, group)
    out = torch.empty((M, N), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_gemm_prepared(dev(case["x"]), qs, dev(case["qzeros"]), dev(case["scales"]), perm, out, group)
    assert_within_band(out.cpu().numpy(), ref, f"repacked M={M} K={K} N={N} g={group}")


def test_repacked_one_hot_rows_are_bit_exact(B):
    K, N, group, M = 512, 136, 128, 4
    case = workloads.make_case(M, K, N, group, seed=3, act_order=True)
    ks = [0, 129, 300, 511]
    case["x"] = workloads.one_hot_activations(M, K, ks)
    w_ref = oracle.dequant(case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    qs, perm = _repack(B, case, group)
    out = torch.empty((M, N), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_gemm_prepared(dev(case["x"]), qs, dev(case["qzeros"]), dev(case["scales"]), perm, out, group)
    assert np.array_equal(out.cpu().numpy().view(np.uint16), w_ref.view(np.uint16)[ks])


def test_repack_refuses_unbalanced_or_out_of_range_groups(B):
    K, N, group = 512, 64, 128
    case = workloads.make_case(1, K, N, group, seed=9, act_order=True)
    qw = dev(case["qweight"])
    qs = torch.empty_like(qw)
    perm = torch.empty(K, dtype=torch.int32, device="cuda")
    g = case["g_idx"].copy()
    g[np.flatnonzero(g == 1)[0]] = 0  # group 0 now owns one row too many
    with pytest.raises(B.GptqError) as e:
        B.gptq_w4a16_act_order_prepare(qw, dev(g), qs, perm, group)
    assert e.value.code == -2
    g = case["g_idx"].copy()
    g[5] = K // group
    with pytest.raises(B.GptqError) as e:
        B.gptq_w4a16_act_order_prepare(qw, dev(g), qs, perm, group)
    assert e.value.code == -1


# ------------------------------------------------------------------ format variants

def test_stored_zero_minus_one_checkpoints_convert_once(B):
    """A checkpoint that stores z - 1 (mod 16), converted with shift_zeros(+1), gives the canonical tensors'
    results bit for bit; shifting by -1 afterwards restores the stored words."""
    M, K, N, group = 4, 1024, 264, 128
    case = workloads.make_case(M, K, N, group, seed=31)
    z = oracle.unpack_qzeros(case["qzeros"])
    stored = oracle.pack_qzeros(((z.astype(np.int32) - 1) % 16).astype(np.uint8))
    converted = torch.empty_like(dev(stored))
    B.gptq_w4a16_shift_zeros(dev(stored), converted, 1, group)
    assert np.array_equal(converted.cpu().numpy().view(np.uint32), case["qzeros"].view(np.uint32))
    back = dev(stored).clone()
    B.gptq_w4a16_shift_zeros(converted, back, -1, group)
    assert np.array_equal(back.cpu().numpy().view(np.uint32), stored.view(np.uint32))
    B.gptq_w4a16_shift_zeros(back, back, 17, group)   # in place, delta taken mod 16
    assert np.array_equal(back.cpu().numpy().view(np.uint32), case["qzeros"].view(np.uint32))


@pytest.mark.parametrize("M", [1, 8, 300])
def test_symmetric_checkpoints_are_zero_point_eight(B, M):
    """No qzeros tensor (symmetric quantisation) = every word 0x88888888."""
    K, N, group = 1024, 264, 128
    case = workloads.make_case(M, K, N, group, seed=32)
    case["qzeros"] = np.full_like(case["qzeros"], np.int32(-2004318072))  # 0x88888888
    assert np.all(oracle.unpack_qzeros(case["qzeros"]) == 8)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    assert_within_band(run_gemm(B, case, group), ref, f"symmetric M={M}")


@pytest.mark.parametrize("M", [1, 8, 300])
@pytest.mark.parametrize("group", [32, 64, 1024])
def test_other_group_sizes_including_one_group_per_column(B, M, group):
    K, N = 1024, 264
    case = workloads.make_case(M, K, N, group, seed=33 + group)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    assert_within_band(run_gemm(B, case, group), ref, f"group={group} M={M}")


# ------------------------------------------------------------------ HIP graph replay

@pytest.mark.parametrize("M,K,N,plan_args", [
    (1, 2816, 520, dict(kernel=1, split_k=4, tile=32)),   # vector kernel, K slices through scratch
    (8, 2048, 328, dict(kernel=3, split_k=3)),            # small-batch MFMA kernel, K slices
    (96, 1408, 288, dict(kernel=2, tile=5, split_k=3)),   # big-tile kernel, K slices
    (48, 1408, 288, dict(kernel=4, split_k=3)),           # mid-batch streaming kernel, K slices
    (1, 1024, 264, dict()),                                # default dispatch
])
def test_graph_replays_match_eager(B, M, K, N, plan_args):
    """A captured launch replayed several times, with eager launches of other problems (which use the same
    scratch and arrival counters) and synchronisations in between, gives the eager result bit for bit every time."""
    group = 128
    case = workloads.make_case(M, K, N, group, seed=M + K + N)
    other = workloads.make_case(3, 1024, 520, group, seed=99)
    plan = B.Plan(**plan_args) if plan_args else None
    eager = run_gemm(B, case, group, plan)
    x, qw, qz, sc = (dev(case[k]) for k in ("x", "qweight", "qzeros", "scales"))
    out = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        B.gptq_w4a16_gemm(x, qw, qz, sc, None, out, group, plan)  # sizes the scratch before capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.gptq_w4a16_gemm(x, qw, qz, sc, None, out, group, plan)
        for rep in range(4):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            got = out.cpu().numpy()
            assert np.array_equal(got.view(np.uint16), eager.view(np.uint16)), f"replay {rep} differs from eager"
            run_gemm(B, other, group, B.Plan(kernel=1, split_k=2, tile=64))  # eager work between the replays


def test_captured_graph_survives_scratch_growth(B):
    """A graph captured on library-owned scratch keeps replaying correctly after a larger eager problem has made
    the library move to a bigger block (the outgrown block is retired, not freed)."""
    group = 128
    B.gptq_w4a16_set_workspace(None)  # back to a fresh library-owned block of minimum size (8 MiB)
    small = workloads.make_case(1, 11008, 4096, group, seed=31)
    assert B.gptq_w4a16_plan_query(1, 11008, 4096, group).split_k > 1
    eager = run_gemm(B, small, group)
    x, qw, qz, sc = (dev(small[k]) for k in ("x", "qweight", "qzeros", "scales"))
    out = torch.zeros((1, 4096), dtype=torch.float16, device="cuda")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.gptq_w4a16_gemm(x, qw, qz, sc, None, out, group)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint16), eager.view(np.uint16))
        # 5 K slices x 96 tiles x 64 x 128 fp32 = 15.7 MB of partial sums: more than the first block holds
        big_plan = B.Plan(kernel=2, tile=5, split_k=5)
        assert B.gptq_w4a16_plan_query(64, 4096, 12288, group, False, big_plan).split_k == 5
        big = workloads.make_case(64, 4096, 12288, group, seed=32)
        run_gemm(B, big, group, big_plan)
        junk = torch.full((16 << 20,), -1, dtype=torch.int32, device="cuda")  # would land in a freed block
        for rep in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().view(np.uint16), eager.view(np.uint16)), f"replay {rep} after growth"
            run_gemm(B, big, group, big_plan)
        del junk


def test_scratch_growth_is_refused_under_capture(B):
    group = 128
    B.gptq_w4a16_set_workspace(None)
    run_gemm(B, workloads.make_case(1, 1024, 264, group, seed=1), group)  # first block: 8 MiB
    big = workloads.make_case(64, 4096, 12288, group, seed=32)
    big_plan = B.Plan(kernel=2, tile=5, split_k=5)  # 15.7 MB of partial sums
    x, qw, qz, sc = (dev(big[k]) for k in ("x", "qweight", "qzeros", "scales"))
    out = torch.zeros((64, 12288), dtype=torch.float16, device="cuda")
    stream = torch.cuda.Stream()
    code = None
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out.zero_()
            try:
                B.gptq_w4a16_gemm(x, qw, qz, sc, None, out, group, big_plan)
            except B.GptqError as e:
                code = e.code
        torch.cuda.synchronize()
    assert code == -5, "growing the scratch while the stream is captured must be refused"
    got = run_gemm(B, big, group, big_plan)  # eagerly it grows and works
    rng = np.random.default_rng(3)
    mi = rng.integers(0, 64, 256).astype(np.int32)
    ni = rng.integers(0, 12288, 256).astype(np.int32)
    ref = oracle.gemm_ref_sampled(big["x"], big["qweight"], big["qzeros"], big["scales"], None, group, mi, ni)
    assert_within_band(got[mi, ni], ref, "after the refused capture")


def test_act_order_table_too_large_for_lds_falls_back(B):
    """896 groups x 64 columns of (scale, zero) do not fit the vector kernel's LDS: the call must not fail."""
    M, K, N, group = 2, 28672, 64, 32
    assert B.gptq_w4a16_plan_query(M, K, N, group, True).kernel == 2
    case = workloads.make_case(M, K, N, group, seed=5, act_order=True)
    out = run_gemm(B, case, group)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    assert_within_band(out, ref, "act-order, 896 groups")


@pytest.mark.parametrize("M,K,N,plan_args", [
    (1, 4096, 520, dict(kernel=1)),
    (4, 4096, 520, dict(kernel=1)),
    (1, 4096, 520, dict(kernel=1, flags=8)),
    (8, 4096, 520, dict(kernel=1)),
    (8, 4096, 520, dict(kernel=3, tile=64)),
    (24, 4096, 520, dict(kernel=3, tile=64, split_k=4)),
    (8, 2048, 1024, dict(kernel=3, tile=256)),
    (32, 2048, 1024, dict(kernel=3, tile=256, split_k=2)),
    (96, 2048, 520, dict(kernel=2)),
    (48, 2048, 520, dict(kernel=4)),
    (100, 2048, 520, dict(kernel=4, split_k=2)),
])
@pytest.mark.parametrize("kind", ["offset", "outliers", "huge_offset"])
def test_activations_with_large_mean_and_outliers(B, M, K, N, plan_args, kind):
    """Activations with a large common offset or with outliers.

    Two things happen then.  (1) The kernels that apply the group's scale AFTER the contraction (vector kernel
    below eight rows, small-batch kernel) compute sum_k x_k * s * (q_k - z) with the unrounded product, the others
    with the fp16-rounded weight of the dequant definition; the two differ by sum_k x_k * delta_k (delta = the fp16
    rounding error of a weight), which is noise for zero-mean activations and adds up coherently under a common
    offset: each kernel is held to the band around ITS definition of W, both computed here in fp64 from the
    oracle's unpacked fields, and within 3 bands of the other one.  (2) The vector kernel below eight rows
    contracts biased codes and cancels sum_k x_k * bias in fp32, which costs digits in proportion to the 32-k
    sums of x: it is held to offsets of a few tens (the last case, sums of ~20000, is for the other kernels).
    """
    group = 128
    scale_after = plan_args["kernel"] == 3 or (plan_args["kernel"] == 1 and M < 8)
    if kind == "huge_offset" and plan_args["kernel"] == 1 and M < 8:
        pytest.skip("beyond the documented input range of the biased-code arithmetic")
    case = workloads.make_case(M, K, N, group, seed=11 * M + len(kind))
    rng = np.random.default_rng(M + K)
    x = case["x"].astype(np.float32)
    if kind == "offset":
        x = x + 40.0
    elif kind == "outliers":
        mask = rng.random(x.shape) < 0.01
        x = np.where(mask, np.sign(x) * rng.uniform(50.0, 100.0, x.shape), x)
    else:
        x = x * 4.0 + 600.0  # every 128-k sum of x is ~77000: beyond fp16
    case["x"] = x.astype(np.float16)
    out = run_gemm(B, case, group, B.Plan(**plan_args)).astype(np.float64)
    ref_rounded = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
    q = oracle.unpack_qweight(case["qweight"]).astype(np.float64)
    z = np.repeat(oracle.unpack_qzeros(case["qzeros"]).astype(np.float64), group, axis=0)
    w_exact = (q - z) * np.repeat(case["scales"].astype(np.float64), group, axis=0)
    ref_exact = case["x"].astype(np.float64) @ w_exact
    own, other = (ref_exact, ref_rounded) if scale_after else (ref_rounded, ref_exact)
    finite = np.abs(ref_rounded) < 60000.0  # outputs beyond fp16 range are not comparable
    assert finite.mean() > 0.9

    def worst(ref):
        return float((np.abs(out - ref)[finite] / (TOL * np.maximum(1.0, np.abs(ref[finite])))).max())

    assert worst(own) <= 0.5, f"{kind}: err/tol = {worst(own):.3f} against the kernel's own definition of W"
    if kind != "huge_offset":
        assert worst(other) <= 8.0, f"{kind}: err/tol = {worst(other):.3f} against the other definition of W"


@pytest.mark.parametrize("K,N,tile", [(4096, 1000, 64), (4096, 2072, 128), (2048, 520, 32), (8192, 776, 256),
                                      (4096, 1000, 0), (1024, 264, 64)])
def test_single_row_group_level_correction(B, K, N, tile):
    """Unsplit single-row plans whose slice gives every row lane whole 128-k groups run the variant that corrects
    bias and zero point once per group (two pipeline steps per group); others the per-chunk kernel.  Both against
    the oracle, ragged last column tile included, and groups of 256 k."""
    for group in (128, 256):
        case = workloads.make_case(1, K, N, group, seed=K + N + tile + group)
        ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)
        plan = B.Plan(kernel=1, tile=tile, split_k=1) if tile else None
        out = run_gemm(B, case, group, plan)
        assert_within_band(out, ref, f"single row K={K} N={N} tile={tile} g={group}")


# ------------------------------------------------------------------ measurement aids

def test_measurement_aids_run_and_validate_their_arguments(B):
    ops = (torch.rand(1 << 12, device="cuda") * 2.0 - 1.0).half()
    sink = torch.zeros(64, dtype=torch.float32, device="cuda")
    buf = torch.zeros(1 << 20, dtype=torch.int32, device="cuda")
    B.gptq_w4a16_stream_probe(buf, sink.view(torch.int32))
    assert B.gptq_w4a16_mfma_probe(ops, sink, 10) > 0
    for waves in (1, 2, 4):
        for v in (0, 2, 4, 6, 8, 12, 16):
            assert B.gptq_w4a16_issue_probe(ops, sink, 5, v, waves) == 4 * waves * 5 * 4
    torch.cuda.synchronize()
    for v, waves, iters in ((3, 2, 5), (4, 3, 5), (4, 2, 0)):
        with pytest.raises(B.GptqError) as err:
            B.gptq_w4a16_issue_probe(ops, sink, iters, v, waves)
        assert err.value.code == -1
