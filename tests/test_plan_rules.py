"""Host logic of the automatic plans (no device is touched)."""
import ctypes
import os
import random
import subprocess
import time

import pytest


@pytest.fixture(scope="module")
def B():
    from paper_2511_19438_amd import build

    if not os.path.exists(build.LIB_PATH):
        build.build()
    from paper_2511_19438_amd import binding

    return binding


def test_automatic_slices_fit_the_static_scratch_block_and_the_grid(B):
    """Big-tile and act-order plans: partial sums within the 48 MiB of gptq_w4a16_gemm_static, slices of whole stages (none
    empty), and K slices of the 128x256 tile only with a compute unit for every workgroup."""
    tile_dims = {1: (256, 256), 3: (128, 128), 5: (64, 128), 8: (128, 256), 64: (64, 64)}
    rng = random.Random(5)
    for _ in range(400):
        group = rng.choice([32, 64, 128])
        K, N = group * rng.randint(2, 28672 // group), 8 * rng.randint(1, 7168)
        M, act = rng.choice([rng.randint(65, 700), rng.randint(17, 2048)]), rng.random() < 0.3
        pl = B.gptq_w4a16_plan_query(M, K, N, group, act)
        if pl.kernel != 2:
            continue
        bm, bn = tile_dims[pl.tile]
        tiles = -(-M // bm) * -(-N // bn)
        if pl.split_k > 1:
            assert pl.split_k * tiles * bm * bn * 4 <= 48 << 20 or act, (M, K, N, group, act)
            forced = 256 * (K // group) + 4 * K > 159 * 1024  # act-order: table and offsets of one slice exceed the LDS
            assert not act or pl.split_k * M * N * 4 <= 48 << 20 or forced, (M, K, N, group)
            stages = -(-K // (128 if act else 64))
            per = -(-stages // pl.split_k)
            assert (pl.split_k - 1) * per < stages, (M, K, N, pl.split_k)
        if pl.tile == 8 and pl.split_k > 1:
            assert tiles * pl.split_k <= 256, (M, K, N, pl.split_k)
            assert B.gptq_w4a16_workspace_bytes(M, K, N, group) >= pl.split_k * tiles * bm * bn * 4


def fields(plan):
    return plan.kernel, plan.split_k, plan.tile, plan.flags


def test_a_queried_plan_given_back_resolves_to_itself(B):
    """Every automatic plan is a valid request for itself, act-order lookups (flag 16) among them."""
    rng = random.Random(11)
    lookups = 0
    for _ in range(2000):
        group = rng.choice([8, 16, 32, 64, 96, 128, 256])
        K, N = group * rng.randint(1, 28672 // group), 8 * rng.randint(1, 4000)
        M, act = int(2 ** rng.uniform(0, 11)), rng.random() < 0.5
        auto = B.gptq_w4a16_plan_query(M, K, N, group, act)
        again = B.gptq_w4a16_plan_query(M, K, N, group, act, auto)
        assert fields(again) == fields(auto), (M, K, N, group, act, fields(auto), fields(again))
        lookups += auto.flags == 16
        assert auto.flags == 0 or act
    assert lookups > 300


def test_the_act_order_lookup_flag_is_refused_where_there_is_no_such_variant(B):
    def code(plan, M=8, K=1024, act=True, group=128):
        try:
            B.gptq_w4a16_plan_query(M, K, 264, group, act, plan)
        except B.GptqError as e:
            return e.code
        return 0

    assert [code(B.Plan(kernel=k, flags=16)) for k in (0, 1, 2, 3, 4)] == [-1, 0, 0, -1, -1]
    assert [code(B.Plan(kernel=2, tile=t, flags=16)) for t in (0, 3, 64, 128)] == [0, -1, 0, -1]
    assert code(B.Plan(kernel=2, tile=64)) == -1 and code(B.Plan(kernel=1, flags=17)) == -1
    assert code(B.Plan(kernel=1, flags=16), act=False) == -1
    assert code(B.Plan(kernel=1, flags=16), M=1) == -2
    assert code(B.Plan(kernel=2, flags=16), K=1032, group=8) == -2   # K % 32
    assert code(B.Plan(kernel=2, flags=16), K=28672, group=32) == -2  # 896 groups do not fit the LDS
    # without the flag the named kernels themselves
    assert fields(B.gptq_w4a16_plan_query(8, 4096, 4096, 128, True, B.Plan(kernel=1)))[3] == 0
    assert fields(B.gptq_w4a16_plan_query(40, 4096, 4096, 128, True, B.Plan(kernel=2)))[2:] == (3, 0)


def test_three_and_four_rows_on_a_k_that_ends_inside_a_unit(B):
    """The faster of the vector kernel (1) and the small-batch kernel (3) at sizes where they measured 10 % and more apart."""
    vector = [(12320, 18432, 32), (8224, 9216, 32), (8224, 16392, 32), (16416, 24576, 32), (28704, 6400, 32), (4128, 20480, 32),
              (28704, 28672, 32), (12352, 18432, 64), (16448, 9216, 64), (28736, 4168, 64), (8256, 24576, 64), (2112, 57344, 32), (2592, 18432, 32), (3136, 17408, 64)]
    small = [(8224, 2056, 32), (28704, 3072, 32), (4128, 4168, 32), (4128, 12288, 32), (6176, 5120, 32), (8224, 6912, 32),
             (4160, 24576, 64), (8256, 4168, 64), (28736, 5120, 64), (2112, 16384, 64), (6208, 28672, 64), (12352, 2304, 64), (704, 21504, 64), (1120, 18432, 32), (1088, 20480, 64)]
    for M in (3, 4):
        assert [s for s in vector if B.gptq_w4a16_plan_query(M, s[0], s[1], s[2]).kernel != 1] == []
        assert [s for s in small if B.gptq_w4a16_plan_query(M, s[0], s[1], s[2]).kernel != 3] == []
    assert all(B.gptq_w4a16_plan_query(5, *s).kernel == 3 for s in vector + small)


def test_deep_layers_at_65_to_96_rows(B):
    """The big-tile kernel (2) only where the layer is wide enough for its tiles; sizes where both measured 5 % and more apart."""
    mid = [(16384, 2048), (16384, 4096), (20480, 5120), (24576, 2048), (24576, 5120), (28672, 4096), (12288, 4096)]
    big = [(18432, 8192), (20480, 12288), (28672, 8192), (24576, 7168), (28672, 6144), (16384, 10240), (28672, 16384)]
    for M in (65, 77, 96):
        assert [s for s in mid if B.gptq_w4a16_plan_query(M, *s, 128).kernel != 4] == []
        assert [s for s in big if B.gptq_w4a16_plan_query(M, *s, 128).kernel != 2] == []
    assert B.gptq_w4a16_plan_query(97, 28672, 8192, 128).kernel == 4
    assert [B.gptq_w4a16_plan_query(M, 20480, 512, 128).kernel for M in (65, 96, 97)] == [2, 2, 4]
    assert [B.gptq_w4a16_plan_query(M, 20480, 640, 128).kernel for M in (65, 80, 81, 96)] == [4, 4, 2, 2]


def test_scratch_of_act_order_slices_is_bounded(B):
    """Slices that the LDS calls for (606 groups: ten of them) ask for no scratch beyond the static block."""
    for M in (64, 200, 512, 2048, 8192):
        for N in (4096, 8192, 28672):
            assert B.gptq_w4a16_plan_query(M, 19392, N, 32, True).split_k == 10
            assert B.gptq_w4a16_workspace_bytes(M, 19392, N, 32) <= 48 << 20, (M, N)


def test_act_order_lookups_serve_as_many_groups_as_the_lds_holds(B):
    flags = lambda M, groups: B.gptq_w4a16_plan_query(M, 32 * groups, 4096, 32, True).flags
    assert [flags(M, 606) for M in (2, 16, 384, 385, 2048)] == [16] * 5
    assert [flags(M, 630) for M in (2, 16, 17, 384, 385)] == [16, 16, 16, 16, 0]
    assert [flags(M, 631) for M in (2, 17, 384)] == [0, 0, 0]


def test_nine_to_sixteen_rows_of_formats_without_a_small_batch_kernel(B):
    """The vector kernel (1) on deep narrow layers, the big-tile kernel (2) elsewhere; sizes measured 8 % and more apart."""
    for M in (9, 11, 16):
        assert {B.gptq_w4a16_plan_query(M, *s, 96).kernel for s in [(8064, 256), (8064, 1024), (12096, 512), (16128, 512), (24192, 256)]} == {1}
        assert {B.gptq_w4a16_plan_query(M, *s, 96).kernel for s in [(4032, 512), (2016, 4096), (8064, 3072), (12096, 1536), (24192, 1024)]} == {2}
    assert B.gptq_w4a16_plan_query(17, 8064, 256, 96).kernel == 2


def test_the_largest_tile_only_where_it_is_the_fastest(B):
    """256x256 (1) or 128x256 (8), sizes where they measured 2 % and more apart."""
    tile = lambda *q: B.gptq_w4a16_plan_query(*q, 128).tile
    assert [tile(*q) for q in [(777, 4096, 12288), (777, 8192, 10240), (129, 8192, 57344), (777, 8192, 57344), (1024, 8192, 57344),
                               (1396, 6656, 26112), (4096, 8192, 10240)]] == [8] * 7
    assert [tile(*q) for q in [(2048, 8192, 57344), (512, 4096, 22016), (2048, 4096, 22016)]] == [1] * 3


def test_act_order_on_a_shallow_k(B):
    """Lookups (flag 16) or the general path; sizes measured 8 % and more apart."""
    flags = lambda M, K, N: B.gptq_w4a16_plan_query(M, K, N, 32, True).flags
    assert [flags(*s) for s in [(64, 256, 40960), (256, 256, 4096), (512, 256, 4096), (512, 544, 4096), (256, 544, 40960),
                                (2048, 768, 16384), (8, 256, 57344)]] == [16] * 7
    assert [flags(*s) for s in [(1024, 256, 4096), (256, 256, 16384), (2048, 256, 40960), (1024, 544, 16384), (2048, 544, 40960)]] == [0] * 5
    assert B.gptq_w4a16_plan_query(2048, 256, 40960, 32, True, B.Plan(kernel=2, flags=16)).flags == 16  # still on request


def test_column_tiles_of_sliced_plans_have_an_arrival_counter_each(B):
    """65536 counters; a width of 32 columns, asked for or chosen, would have more tiles beyond 2097152 columns."""
    for M in (2, 16, 24, 32):
        for N in (2097152, 2097160, 2097168, 3000000, 4194304):
            for plan in (dict(kernel=3, tile=32), dict(kernel=4, tile=32), dict(kernel=3), dict(kernel=4)):
                for split in (0, 1, 2):
                    pl = B.gptq_w4a16_plan_query(M, 256, N, 128, False, B.Plan(split_k=split, **plan))
                    assert split == 0 or pl.split_k == split
                    assert pl.split_k == 1 or -(-N // pl.tile) <= 65536, (M, N, plan, pl.tile)
    # what can be had is taken as asked: the last width with a counter for every tile, and any width without slices
    assert B.gptq_w4a16_plan_query(2, 256, 2097152, 128, False, B.Plan(kernel=3, tile=32, split_k=2)).tile == 32
    assert B.gptq_w4a16_plan_query(2, 256, 2097160, 128, False, B.Plan(kernel=3, tile=32, split_k=1)).tile == 32
    # beyond it the width is chosen, as for any other that does not exist
    for M in (2, 24):
        for kernel in (3, 4):
            asked, auto = (B.gptq_w4a16_plan_query(M, 256, 2097160, 128, False, B.Plan(kernel=kernel, tile=t, split_k=2)) for t in (32, 0))
            assert kernel == 4 or fields(asked) == fields(auto)


def test_automatic_slices_of_the_ring_have_a_compute_unit_each(B):
    """Eight wavefronts add the sums of an automatic slice up, as they do where there is no scratch for the slices: whatever
    width a plan names, under either kernel's id.  A number of slices that a plan names is its own."""
    rng = random.Random(17)
    sliced = 0
    for _ in range(1500):
        group = rng.choice([32, 64, 128])
        M, K, N = rng.randint(1, 32), 128 * rng.randint(8, 224), 8 * rng.randint(64, 2048)
        kernel, tile = rng.choice([3, 4]), rng.choice([0, 32, 64, 96, 128])
        pl = B.gptq_w4a16_plan_query(M, K, N, group, False, B.Plan(kernel=kernel, tile=tile))
        if pl.kernel not in (3, 4) or pl.tile == 256:
            continue  # (a format or a width of other kernels)
        assert pl.split_k == 1 or pl.split_k * -(-N // pl.tile) <= 256, (M, K, N, group, kernel, tile, pl.tile, pl.split_k)
        sliced += pl.split_k > 1
    assert sliced > 300
    pl = B.gptq_w4a16_plan_query(24, 8192, 4096, 128, False, B.Plan(kernel=4, tile=32, split_k=4))
    assert (pl.kernel, pl.tile, pl.split_k) == (4, 32, 4)


def test_small_batches_on_deep_narrow_layers(B):
    """Narrow tiles, which measured 10 % and more ahead of ten and more slices of 96 and 128 columns at these sizes."""
    for K, N, group in [(9472, 1792, 128), (11392, 1664, 128), (10112, 2048, 64), (12288, 1600, 32), (24704, 1792, 64),
                        (21888, 2464, 128), (9344, 1792, 32), (25728, 1792, 128), (14336, 1456, 64), (23552, 1792, 128)]:
        pl = B.gptq_w4a16_plan_query(2, K, N, group)
        assert pl.kernel == 3 and pl.tile <= 64, (K, N, group, pl.tile, pl.split_k)


def test_small_tiles_of_small_groups(B):
    """The plan of the big-tile kernel with groups of 32 where it measured 8-15 % ahead of the one that another pace of two
    wavefront groups would give.  (174x2496x15488: 128x256 in two slices 30.0 us, which was ahead of the tiles there were then;
    two of 96x128 unsplit 24.7.)"""
    plan = lambda M, K, N: (lambda pl: (pl.kernel, pl.tile, pl.split_k))(B.gptq_w4a16_plan_query(M, K, N, 32))  # noqa: E731
    for problem, want in {(202, 7200, 2040): (5, 4), (174, 2496, 15488): (5, 1), (158, 2976, 10880): (5, 1), (378, 2112, 9064): (3, 1),
                          (558, 2368, 1352): (5, 2), (424, 5056, 1408): (5, 3), (678, 4480, 2048): (5, 4), (357, 3200, 10496): (3, 1)}.items():
        assert plan(*problem) == (2, *want), problem


def test_slices_asked_for_up_to_128_rows_leave_the_largest_tile_out(B):
    """256x256 has no rows for them; a plan that names it still gets it, and one under the mid-batch kernel's id, which has no
    such tile, resolves to itself."""
    for M, K, N, group, split in [(128, 8192, 8192, 128, 8), (113, 2432, 14080, 128, 4), (69, 3040, 5888, 32, 8), (31, 2944, 1536, 128, 16)]:
        for kernel in (0, 2, 4):
            pl = B.gptq_w4a16_plan_query(M, K, N, group, False, B.Plan(kernel=kernel, split_k=split))
            assert pl.tile != 1, (M, K, N, kernel)
            assert fields(B.gptq_w4a16_plan_query(M, K, N, group, False, pl)) == fields(pl), (M, K, N, kernel)
        assert B.gptq_w4a16_plan_query(M, K, N, group, False, B.Plan(kernel=2, tile=1, split_k=split)).tile == 1


def test_slices_and_tiles_asked_for_without_a_kernel(B):
    """A plan that leaves the kernel open gets the slices and the tile that it names all the same, whichever kernel runs under
    the mid-batch kernel's id (its own, the ring up to 64 rows, the big-tile kernel from 49 on), and resolves to itself."""
    kernels = set()
    for M, K, N, group in [(24, 4096, 22016, 128), (24, 28672, 8192, 64), (32, 8192, 57344, 128), (33, 8192, 1024, 64), (40, 11008, 4096, 128),
                           (48, 8192, 1024, 128), (48, 4032, 4096, 64), (56, 8192, 1024, 128), (56, 11008, 4096, 128), (64, 8192, 10240, 128),
                           (64, 4096, 4096, 128), (64, 24960, 17344, 128), (77, 8192, 10240, 128), (100, 11008, 4096, 64), (128, 8192, 8192, 128)]:
        assert B.gptq_w4a16_plan_query(M, K, N, group).kernel == 4
        for split in (1, 2, 3, 4, 5, 8):
            asked = B.gptq_w4a16_plan_query(M, K, N, group, False, B.Plan(split_k=split))
            assert asked.kernel == 4 and asked.split_k == split, (M, K, N, split, fields(asked))
            assert fields(B.gptq_w4a16_plan_query(M, K, N, group, False, asked)) == fields(asked), (M, K, N, split)
            kernels.add(asked.tile)
        for tile in (32, 64, 96, 128, 3, 5, 8):
            named, asked = (B.gptq_w4a16_plan_query(M, K, N, group, False, B.Plan(kernel=k, tile=tile, split_k=2)) for k in (4, 0))
            if named.tile == tile:  # (a tile that one of the kernels has at these rows)
                assert fields(asked) == fields(named), (M, K, N, tile, fields(asked), fields(named))
                assert B.gptq_w4a16_plan_query(M, K, N, group, False, B.Plan(tile=tile)).tile == tile, (M, K, N, tile)
    assert kernels >= {32, 64, 128, 5, 8}


def test_planning_stays_short_where_several_kernels_are_weighed(B):
    """49-64 rows weigh the mid-batch kernel against the big-tile kernel, whose plan has four numbers of rows to a workgroup
    there: a lone call waits for that on the host.  In units of the ring's search for 32 rows: 2.4 (searching twice, and every
    estimate from the problem's sizes on, it was 13)."""
    lib, out = B.load(), B.Plan()
    named = B.Plan(kernel=4, tile=64)  # (names everything: a call without a search)
    calls = [(100, 8192, 10240, ctypes.byref(named)), (32, 4096, 4096, None), (56, 8192, 10240, None), (64, 24960, 17344, None), (77, 8192, 10240, None)]
    best = [1e9] * len(calls)
    for attempt in range(2000):  # (in turn, the shortest of each: whatever else the machine does; more turns where that did not do)
        for i, (M, K, N, request) in enumerate(calls):
            start = time.perf_counter()
            for _ in range(100):
                lib.gptq_w4a16_plan_query(M, K, N, 128, 0, request, ctypes.byref(out))
            best[i] = min(best[i], time.perf_counter() - start)
        alone, ring, *searches = best
        if attempt >= 40 and max(searches) - alone <= 5 * (ring - alone):
            return
    raise AssertionError([b * 1e4 for b in best])


PLANNER = r"""
#include "prefill.hip"
namespace gptq {
namespace prefill {
#define NO_DEVICE(tile) template <> hipError_t launch_tile<tile>(const Args &, int, int, hipStream_t) { return hipErrorNoDevice; }
%s
}  // namespace prefill
}  // namespace gptq
extern "C" __attribute__((visibility("default"))) void plan(int M, int K, int N, int group, int tile, int split, int *out)
{
    gptq::Problem p = {};
    p.M = M, p.K = K, p.N = N, p.group_size = group;
    gptq::PrefillPlan plan = {tile, split, 0, false};
    gptq::prefill_make_plan(p, plan);
    out[0] = plan.rows;
    out[1] = gptq::k_groups(plan.tile, gptq::grid_of(p, plan.tile, plan.rows), gptq::slices_of(p, plan.split_k));
    out[2] = gptq::mode_of(p) == gptq::prefill::kGroupPerHalf;
}
"""


def test_the_problems_of_the_gpu_tests_get_the_rows_that_they_are_for(tmp_path):
    """The rows to a workgroup and the wavefront groups are no part of a plan query: the host code of the big-tile kernel on its own."""
    from paper_2511_19438_amd import build
    from tests.test_gpu_two_groups import ROWS_THAT_FIT

    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    source, lib = tmp_path / "planner.hip", tmp_path / "planner.so"
    source.write_text(PLANNER % "\n".join(f"NO_DEVICE({t})" for t in build.PREFILL_TILES))
    flags = [f for f in build.COMMON if f != "-fvisibility=hidden"]
    proc = subprocess.run([build.HIPCC, *flags, "--cuda-host-only", "-shared", str(source), "-o", str(lib)], capture_output=True, text=True)
    assert proc.returncode == 0, proc.stderr[-2000:]
    plan, out = ctypes.CDLL(str(lib)).plan, (ctypes.c_int * 3)()
    seen = set()
    for tile, M, K, N, group, split, rows, groups in ROWS_THAT_FIT:
        plan(M, K, N, group, tile, split, out)
        assert tuple(out)[:2] == (rows, groups), (tile, M, K, N, group, split)
        seen.add((tile, rows, groups, bool(out[2])))
    assert seen >= {(t, r, g, h) for t in (5, 8) for r in (80, 96, 112) for g in (1, 2) for h in (False, True)}
