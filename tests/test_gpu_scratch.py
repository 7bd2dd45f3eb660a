"""What a call does where the scratch of its K slices cannot be had (GPU): a caller's workspace that is too small, growth
while the stream is captured, the static block.  Bars as in test_gpu_parity.py."""
import contextlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2511_19438_amd import workloads  # noqa: E402
from test_gpu_parity import B, _repack, assert_within_band, dev, run_gemm  # noqa: E402,F401

COUNTERS = 1 << 18  # the arrival counters alone


@contextlib.contextmanager
def workspace(B, nbytes):
    buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")  # (borrowed by the library: it has to live as long)
    B.gptq_w4a16_set_workspace(buf)
    try:
        yield buf
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


def vector_scratch(B, M, K, N, group, act):
    """What the vector kernel takes for a batch of up to 16 rows (the least that an automatic call of so few asks for)."""
    plan = B.gptq_w4a16_plan_query(M, K, N, group, act, B.Plan(kernel=1))
    return COUNTERS + (plan.split_k * M * N * 4 if plan.kernel == 1 and plan.split_k > 1 else 0)


# small groups or a width of 8 mod 32 on every tile, with and without two wavefront groups, a K that ends half-way through
# a stage, 96 and 128 rows; act-order from two rows to several row tiles, with a K that ends inside a unit
@pytest.mark.parametrize("M,K,N,group,act,tile", [
    (300, 4096, 1024, 128, False, 0), (200, 2048, 544, 64, False, 3), (150, 2560, 512, 128, False, 8), (77, 4096, 512, 128, False, 8),
    (100, 2304, 8, 128, False, 0), (108, 1056, 32, 96, False, 0), (143, 928, 16, 32, False, 0),
    (359, 640, 8, 128, False, 3), (40, 4256, 136, 32, False, 3), (40, 4256, 136, 32, False, 5),
    (52, 1408, 104, 128, False, 8), (100, 2304, 264, 96, False, 8), (206, 1440, 16, 160, False, 8),
    (45, 3072, 264, 32, False, 8), (70, 4256, 40, 32, False, 8), (286, 7296, 1032, 128, False, 0),
    (12, 2112, 1032, 96, False, 0), (2, 768, 8704, 128, True, 0), (11, 704, 10416, 32, True, 0),
    (32, 2752, 1032, 32, False, 0), (17, 1120, 520, 32, False, 0), (24, 4128, 264, 32, False, 0), (32, 4160, 264, 64, False, 0),
    (11, 704, 2056, 64, False, 0), (3, 3552, 6960, 32, False, 0), (5, 4160, 264, 32, False, 0),
    (24, 2048, 264, 128, True, 0), (40, 2208, 520, 96, True, 0), (130, 2144, 72, 8, True, 0), (300, 4096, 264, 128, True, 0)])
def test_the_result_does_not_depend_on_the_scratch(B, M, K, N, group, act, tile):
    case = workloads.make_case(M, K, N, group, seed=M + N, act_order=act)
    plan = B.Plan(kernel=2, tile=tile) if tile else None
    resolved = B.gptq_w4a16_plan_query(M, K, N, group, act, plan)
    assert resolved.kernel == (3 if not act and group in (32, 64) and M <= 32 else resolved.kernel if act else 2)
    assert resolved.split_k > 1 or resolved.kernel == 3  # (the small-batch kernel asks for its counters all the same)
    sliced = run_gemm(B, case, group, plan)
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    assert_within_band(sliced, ref, "slices in parallel")
    with workspace(B, vector_scratch(B, M, K, N, group, act) if M <= 16 else COUNTERS):
        assert np.array_equal(bits(run_gemm(B, case, group, plan)), bits(sliced))


@pytest.mark.parametrize("M,K,N,group,act", [(40, 4256, 136, 32, False), (300, 2016, 264, 96, False), (40, 2048, 264, 128, True),
                                             (32, 2752, 1032, 32, False), (32, 1120, 520, 32, False)])
def test_a_call_captured_before_there_is_scratch_gives_the_same_bits(B, M, K, N, group, act):
    case = workloads.make_case(M, K, N, group, seed=M, act_order=act)
    resolved = B.gptq_w4a16_plan_query(M, K, N, group, act)
    assert resolved.split_k > 1 or resolved.kernel == 3  # (as above)
    eager = run_gemm(B, case, group)
    x, qw, qz, sc, gi = (dev(case[k]) for k in ("x", "qweight", "qzeros", "scales", "g_idx"))
    out = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    torch.cuda.synchronize()
    B.gptq_w4a16_set_workspace(None)  # the library owns no scratch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.gptq_w4a16_gemm(x, qw, qz, sc, gi, out, group)
        for rep in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(bits(out.cpu().numpy()), bits(eager)), f"replay {rep}"
            assert np.array_equal(bits(run_gemm(B, case, group)), bits(eager))  # eagerly, on scratch of its own


def test_static_act_order_beyond_its_block_gives_the_bits_of_the_regular_call(B):
    """606 groups leave the LDS no room for longer slices: ten of them, whose partial sums exceed the static block."""
    M, K, N, group = 320, 19392, 4096, 32
    plan = B.gptq_w4a16_plan_query(M, K, N, group, True)
    assert plan.split_k * M * N * 4 > 48 << 20
    case = workloads.make_case(M, K, N, group, seed=6, act_order=True)
    x, qw, qz, sc, gi = (dev(case[k]) for k in ("x", "qweight", "qzeros", "scales", "g_idx"))
    out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_gemm_static(x, qw, qz, sc, gi, out, group)
    got = run_gemm(B, case, group)
    assert np.array_equal(bits(out.cpu().numpy()), bits(got))
    mi, ni = workloads.sample_positions(M, N, 256, 3)
    ref = oracle.gemm_ref_sampled(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group, mi, ni)
    assert_within_band(got[mi, ni], ref, "ten slices one after the other")


@pytest.mark.parametrize("M,K,N,group", [(40, 4256, 136, 32), (333, 2752, 1032, 32), (24, 2752, 1032, 32), (100, 2304, 264, 96),
                                         (3, 3552, 6960, 32), (12, 2112, 1032, 96)])
def test_a_repacked_checkpoint_runs_without_the_scratch_of_its_slices(B, M, K, N, group):
    """A workspace that holds the counters and the gathered activations (up to 16 rows: and what the vector kernel takes)."""
    case = workloads.make_case(M, K, N, group, seed=M, act_order=True)
    assert B.gptq_w4a16_plan_query(M, K, N, group).split_k > 1
    qs, perm = _repack(B, case, group)
    x, qz, sc = (dev(case[k]) for k in ("x", "qzeros", "scales"))

    def run():
        out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        return B.gptq_w4a16_gemm_prepared(x, qs, qz, sc, perm, out, group).cpu().numpy()

    sliced = run()
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], case["g_idx"], group)
    assert_within_band(sliced, ref, "slices in parallel")
    least = vector_scratch(B, M, K, N, group, False) if M <= 16 else COUNTERS
    with workspace(B, (least + 255) // 256 * 256 + 2 * M * K):
        assert np.array_equal(bits(run()), bits(sliced))
    with workspace(B, least + 2 * M * K - 256):
        with pytest.raises(B.GptqError) as e:
            run()
        assert e.value.code == -5


def test_a_deep_layer_runs_on_the_workspace_that_served_it_with_fewer_slices(B):
    """The mid-batch kernel's slices took 15 MB here, the big-tile kernel's take 34."""
    M, K, N, group = 77, 28672, 8192, 128
    mid = B.gptq_w4a16_plan_query(M, K, N, group, False, B.Plan(kernel=4))
    assert mid.kernel == 4
    case = workloads.make_case(M, K, N, group, seed=1)
    x, qw, qz, sc = (dev(case[k]) for k in ("x", "qweight", "qzeros", "scales"))
    want, got = (torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    B.gptq_w4a16_gemm(x, qw, qz, sc, None, want, group)
    with workspace(B, COUNTERS + mid.split_k * M * N * 4):
        B.gptq_w4a16_gemm(x, qw, qz, sc, None, got, group)
        torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    mi, ni = workloads.sample_positions(M, N, 128, 2)
    ref = oracle.gemm_ref_sampled(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group, mi, ni)
    assert_within_band(want.cpu().numpy()[mi, ni], ref, "77 rows of a deep layer")


@pytest.mark.parametrize("owned", [True, False])
def test_new_scratch_is_clear_before_another_stream_uses_it(B, owned):
    """The null stream, on which the memory is cleared, is busy; the stream of the call does not wait for it."""
    M, K, N, group = 8, 4096, 1024, 128
    case = workloads.make_case(M, K, N, group, seed=2)
    assert B.gptq_w4a16_plan_query(M, K, N, group).split_k > 1
    want = run_gemm(B, case, group)
    x, qw, qz, sc = (dev(case[k]) for k in ("x", "qweight", "qzeros", "scales"))
    out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    a = torch.randn(8192, 8192, device="cuda").half()
    dirty = torch.full((64 << 20,), 0x5a, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    try:
        for _ in range(5):
            B.gptq_w4a16_set_workspace(None)
            out.fill_(float("nan"))
            dirty.fill_(0x5a)
            torch.cuda.synchronize()
            for _ in range(10):
                a @ a  # about 10 ms on the default (null) stream
            if not owned:
                B.gptq_w4a16_set_workspace(dirty)
            with torch.cuda.stream(torch.cuda.Stream()):
                B.gptq_w4a16_gemm(x, qw, qz, sc, None, out, group)
            torch.cuda.synchronize()
            assert np.array_equal(bits(out.cpu().numpy()), bits(want))
    finally:
        B.gptq_w4a16_set_workspace(None)
