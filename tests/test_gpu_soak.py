"""Bounded soak of the K-slice exchange (GPU): a few thousand launches that cycle through the K-split paths of all
four GEMM kernels over changing shapes, every result compared bit for bit with the first result of its case.

The exchange of partial sums between workgroups rests on write-through stores, an acknowledged-store wait and an
arrival counter (see csrc/exchange.h); a lost or stale partial sum would show as a changed output bit.  The run
stops at the first mismatch and takes well under half a minute.
"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2511_19438_amd import workloads  # noqa: E402

# (M, K, N, act_order, plan fields[, group, 128 if not given]): every plan has K slices
CASES = [
    (1, 4096, 1024, False, dict(kernel=1, tile=64, split_k=4)),
    (4, 2048, 520, False, dict(kernel=1, tile=32, split_k=7)),
    (1, 11008, 4096, False, dict()),                              # the benchmark's down projection, automatic plan
    (2, 1024, 264, True, dict(kernel=1, split_k=2)),
    (8, 4096, 1024, False, dict(kernel=3, tile=64, split_k=4)),
    (24, 2048, 520, False, dict(kernel=3, tile=64, split_k=3)),
    (16, 4096, 4096, False, dict()),                              # small-batch kernel, automatic plan: two slices that swap their sums
    (2, 4096, 520, False, dict(kernel=3, tile=32, split_k=2)),    # the same swap on every width and row count of the ring
    (9, 2048, 1024, False, dict(kernel=3, tile=96, split_k=2)),
    (20, 2048, 264, False, dict(kernel=3, tile=64, split_k=2), 64),
    (32, 4096, 1032, False, dict(kernel=3, tile=128, split_k=2), 32),
    (8, 4096, 2056, False, dict(kernel=3, tile=32, split_k=4)),   # more slices of the ring: through scratch
    (48, 4096, 1024, False, dict(kernel=3, tile=64, split_k=2)),
    (64, 4096, 1024, False, dict(kernel=2, tile=5, split_k=8)),
    (56, 4096, 1024, False, dict(kernel=4, tile=64, split_k=4)),
    (120, 2048, 544, False, dict(kernel=4, split_k=3)),
    (100, 2048, 544, False, dict(kernel=2, tile=3, split_k=2)),
    (64, 4096, 4096, False, dict()),                              # the ring on four row blocks, automatic plan with K slices
    (40, 11008, 520, False, dict()),                              # ... on three, many slices
    (77, 8192, 8192, False, dict()),                              # the big-tile kernel in the mid-batch kernel's place
    (8, 4096, 1024, True, dict()),                                # act-order lookups: one row tile
    (200, 4096, 520, True, dict()),                               # several: a counter per row and column tile
    (120, 2560, 520, False, dict(kernel=2, tile=8, split_k=2)),   # two wavefront groups, half of the threads exchange
    (96, 2560, 520, False, dict(kernel=2, tile=8, split_k=2)),    # the same on 96 rows
    (40, 4256, 136, False, dict(), 32),                           # big-tile kernel with a group row per half stage
    (70, 4256, 520, False, dict(kernel=2, tile=8, split_k=3), 32),
    # the other rows to a workgroup, whose accumulators travel in batches of their own: 80, 96 and 112 of 128 columns, 80 and 112 of 256
    (80, 3392, 5216, False, dict(kernel=2, tile=5), 64),
    (96, 3904, 5152, False, dict(kernel=2, tile=5), 64),
    (95, 1728, 5936, False, dict(kernel=2, tile=5), 96),
    (97, 2912, 8464, False, dict(kernel=2, tile=5), 32),
    (80, 1920, 520, False, dict(kernel=2, tile=8, split_k=3)),
    (112, 1536, 520, False, dict(kernel=2, tile=8, split_k=2), 64),
]
ROUNDS = 1500
BUDGET_S = 25.0


def test_k_split_exchange_soak():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_19438_amd import binding as B

    B.load()
    prepared = []
    for i, (M, K, N, act, plan_args, *rest) in enumerate(CASES):
        group = rest[0] if rest else 128
        plan = B.Plan(**plan_args) if plan_args else None
        resolved = B.gptq_w4a16_plan_query(M, K, N, group, act, plan)
        assert resolved.split_k > 1, f"case {i} is meant to exchange partial sums"
        case = workloads.make_case(M, K, N, group, seed=900 + i, act_order=act)
        dev = {k: (None if v is None else torch.from_numpy(np.ascontiguousarray(v)).cuda()) for k, v in case.items()}
        out = torch.zeros((M, N), dtype=torch.float16, device="cuda")
        B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], dev["g_idx"], out, group, plan)
        torch.cuda.synchronize()
        prepared.append((dev, plan, group, out, out.clone().view(torch.int16)))
    bad = torch.zeros(len(CASES), dtype=torch.int32, device="cuda")
    t0 = time.perf_counter()
    launches = 0
    for rnd in range(ROUNDS):
        for i, (dev, plan, group, out, first) in enumerate(prepared):
            out.fill_(float("nan"))
            B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], dev["g_idx"], out, group, plan)
            bad[i] += (out.view(torch.int16) != first).any().to(torch.int32)
            launches += 1
        if rnd % 20 == 19 or rnd == ROUNDS - 1:
            counts = bad.cpu().numpy()  # synchronises
            assert not counts.any(), f"round {rnd}: outputs changed between launches, per case {counts.tolist()}"
            if time.perf_counter() - t0 > BUDGET_S:
                break
    assert launches >= 20 * len(CASES)
