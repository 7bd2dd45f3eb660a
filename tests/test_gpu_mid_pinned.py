"""The mid-batch kernel's pinned loop (33-96 rows): the edges of its rows, and every remainder of its pipeline."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_19438_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2511_19438_amd import binding
    binding.load()
    return binding


# four wavefronts share K / 64 stages: none, one, two, three (a whole turn of the ring) to eight each, uneven shares
@pytest.mark.parametrize("M,K,N,group,split", [(65, 64, 8, 64, 1), (96, 256, 72, 64, 1), (66, 576, 136, 192, 1), (95, 768, 64, 128, 1),
                                               (80, 1088, 200, 64, 1), (77, 1920, 264, 128, 1), (96, 2048, 520, 256, 3),
                                               (33, 64, 8, 64, 1), (64, 576, 72, 192, 1), (63, 768, 136, 128, 1), (40, 1088, 200, 64, 1),
                                               (33, 6144, 136, 128, 1), (50, 6208, 136, 64, 1), (64, 8192, 8, 128, 1),
                                               (64, 4096, 264, 128, 2), (33, 3968, 136, 128, 2), (48, 1984, 200, 64, 2)])
# (at 33-48 rows 64 columns of whole 128 k are the ring's: 33x6144 and 33x3968 run it, their 128 columns the pinned loop)
# (and stages of a slice on both sides of where 128-column tiles take eight wavefronts on the plain loop)
@pytest.mark.parametrize("tile", [64, 128])
def test_pinned_loop_matches_the_oracle(B, M, K, N, group, split, tile):
    case = workloads.make_case(M, K, N, group, seed=K + M)
    dev = {k: torch.from_numpy(case[k]).cuda() for k in ("x", "qweight", "qzeros", "scales")}
    # an infinite activation reaches its own row alone, and only through the stage that holds it
    dev["x"][M - 1, K - 1] = float("inf")
    out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    B.gptq_w4a16_gemm(dev["x"], dev["qweight"], dev["qzeros"], dev["scales"], None, out, group, B.Plan(kernel=4, split_k=split, tile=tile))
    got = out.cpu().numpy().astype(np.float64)[:M - 1]
    ref = oracle.gemm_ref(case["x"], case["qweight"], case["qzeros"], case["scales"], None, group)[:M - 1]
    assert np.all(np.abs(got - ref) <= 2e-2 * np.maximum(1.0, np.abs(ref)))
    assert not np.isfinite(out[M - 1].float().cpu().numpy()).any()
