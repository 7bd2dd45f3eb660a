"""The workloads that the speed of this library is judged by, from its smallest call to its largest.

A case is one of

  gemm       ``layers`` repetitions of a set of linear layers, each multiplied through ``gptq_w4a16_gemm`` - a decode
             step or a prefill chunk of a model goes through its layers in just this way.  With ``graph`` the calls are
             captured once with ``gptq_w4a16_gemm_static`` and a pass replays the graph, as a serving loop does for
             single-row decoding (``bench.py`` measures its decode step alike).
  act_order  one act-order checkpoint multiplied as it is stored (``g_idx`` passed to ``gptq_w4a16_gemm``).
  repacked   the same checkpoint after the one-time ``gptq_w4a16_act_order_prepare``.
  dequant    the fp16 weights themselves (export, or a dense library product afterwards).

Every layer of a case has weights of its own: the sets of several layers exceed the 256 MB memory-side cache, so that
a pass streams them from HBM as a model's pass does.  Codes, zero points and scales have the distributions of
``paper_2511_19438_amd.workloads``; inputs are drawn on the GPU from the seed.
"""
import math

import torch

from paper_2511_19438_amd import binding
from paper_2511_19438_amd.workloads import ACT_ORDER_SHAPE, LLAMA_7B, LLAMA_70B

SETS = {"llama7b": [(s.K, s.N) for s in LLAMA_7B], "llama70b": [(s.K, s.N) for s in LLAMA_70B]}


def _case(name, op, m, shapes, group=128, layers=1, graph=False):
    case = {"op": op, "m": m, "shapes": shapes, "group": group, "layers": layers, "graph": graph}
    return dict({"name": name}, **case) if name else case


def listed():
    act = f"{ACT_ORDER_SHAPE.K}x{ACT_ORDER_SHAPE.N}"
    return [
        # the smallest call: one row through one attention output projection, where launch and latency count
        _case("call_m1", "gemm", 1, "4096x4096"),
        # single-stream decoding: eight layers of the 7B set in a HIP graph (the serving loop of bench.py)
        _case("decode_7b_m1", "gemm", 1, "llama7b", layers=8, graph=True),
        # single-stream decoding of the 70B set, two layers, called eagerly
        _case("decode_70b_m1", "gemm", 1, "llama70b", layers=2),
        # a decode step of eight streams
        _case("decode_7b_m8", "gemm", 8, "llama7b", layers=8),
        # a decode step of the batch of 32 prompts that the method was evaluated with
        _case("decode_7b_m32", "gemm", 32, "llama7b", layers=8),
        # a larger, odd batch: continuous batching rarely has a round number of streams
        _case("decode_70b_m77", "gemm", 77, "llama70b", layers=2),
        # prefill in chunks of 512 tokens, one layer
        _case("prefill_7b_m512", "gemm", 512, "llama7b"),
        # the largest: 2048 tokens of prefill through one layer of the 70B set
        _case("prefill_70b_m2048", "gemm", 2048, "llama70b"),
        # an act-order checkpoint as stored, eight streams
        _case("act_order_m8", "act_order", 8, act),
        # the same kind of checkpoint after its one-time repack, sixteen streams
        _case("repacked_m16", "repacked", 16, act),
        # a ragged prompt on a layer with small groups whose width is no multiple of a tile
        _case("ragged_g32_m333", "gemm", 333, "2752x6888", group=32),
        # a whole layer's weights dequantised
        _case("dequant", "dequant", 0, "11008x4096"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: batch 1..2048, K 1024..28672, N 1024..57344, groups of 32, 64 and 128, every operation."""
    op = rng.choice(["gemm"] * 7 + ["act_order", "repacked", "dequant"])
    m = _log_int(rng, 1, 2048) if rng.random() < 0.6 else rng.choice([1, 1, 2, 4, 8, 16, 32, 64, 128, 512, 2048])
    if op == "gemm" and rng.random() < 0.25:
        model = rng.choice(["llama7b", "llama7b", "llama70b"])
        layers = rng.randint(2, 8) if model == "llama7b" else rng.randint(1, 2)
        if m > 64:
            layers = 1  # keeps the cost under the largest listed case
        return _case(None, op, m, model, layers=layers, graph=(m <= 8 and rng.random() < 0.5))
    group = rng.choice([128, 128, 128, 64, 32])
    most = 8192 * 57344
    if op == "act_order":
        m = min(m, 512)
        most = 1 << 26  # per-row lookups: larger ones would outlast the largest listed case
    while True:
        k = max(1, round(_log_int(rng, 1024, 28672) / group)) * group
        n = max(1, round(_log_int(rng, 1024, 57344) / 8)) * 8
        if rng.random() < 0.5:
            n = max(1, round(n / 128)) * 128
        if k * n > most:
            continue
        if (group < 64 or n % 32) and m * k * n > 1 << 38:
            continue
        break
    return _case(None, op, 0 if op == "dequant" else m, f"{k}x{n}", group=group)


def _shapes(case):
    if case["shapes"] in SETS:
        return SETS[case["shapes"]] * case["layers"]
    k, n = case["shapes"].split("x")
    return [(int(k), int(n))] * case["layers"]


def _words(rows, cols, gen):
    return torch.randint(-2 ** 31, 2 ** 31, (rows, cols), dtype=torch.int32, device="cuda", generator=gen)


def prepare(case, seed):
    """Weights in the checkpoint format, activations and output buffers; the repack or the graph where the case has one."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    m, group = case["m"], case["group"]
    calls = []
    acts = {}  # layers of one width share their input, as the projections of a layer do
    for k, n in _shapes(case):
        weights = {"qweight": _words(k // 8, n, gen), "qzeros": _words(k // group, n // 8, gen),
                   "scales": torch.empty(k // group, n, device="cuda").uniform_(0.001, 0.01, generator=gen).half()}
        if case["op"] == "dequant":
            calls.append(dict(weights, out=torch.empty(k, n, dtype=torch.float16, device="cuda")))
            continue
        if k not in acts:
            acts[k] = torch.randn(m, k, device="cuda", generator=gen).half()
        call = dict(weights, x=acts[k], out=torch.empty(m, n, dtype=torch.float16, device="cuda"), g_idx=None)
        if case["op"] != "gemm":
            perm = torch.randperm(k, device="cuda", generator=gen)
            call["g_idx"] = (perm // group).to(torch.int32)
        if case["op"] == "repacked":
            qweight, order = torch.empty_like(call["qweight"]), torch.empty(k, dtype=torch.int32, device="cuda")
            binding.gptq_w4a16_act_order_prepare(call["qweight"], call["g_idx"], qweight, order, group)
            call.update(qweight=qweight, order=order)
        calls.append(call)
    state = {"op": case["op"], "group": group, "calls": calls, "outs": [c["out"] for c in calls], "graph": None}
    if case["graph"]:
        _step_static(state)  # once eagerly, as a program does before it captures
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _step_static(state)
        for out in state["outs"]:
            out.zero_()
        state["graph"] = graph
    return state


def _step_static(state):
    group = state["group"]
    for c in state["calls"]:
        binding.gptq_w4a16_gemm_static(c["x"], c["qweight"], c["qzeros"], c["scales"], c["g_idx"], c["out"], group)


def run(state):
    op, group = state["op"], state["group"]
    if state["graph"] is not None:
        state["graph"].replay()
    elif op == "dequant":
        for c in state["calls"]:
            binding.gptq_w4a16_dequant(c["qweight"], c["qzeros"], c["scales"], None, c["out"], group)
    elif op == "repacked":
        for c in state["calls"]:
            binding.gptq_w4a16_gemm_prepared(c["x"], c["qweight"], c["qzeros"], c["scales"], c["order"], c["out"],
                                             group)
    else:
        for c in state["calls"]:
            binding.gptq_w4a16_gemm(c["x"], c["qweight"], c["qzeros"], c["scales"], c["g_idx"], c["out"], group)
    return state["outs"]


def work(case):
    """Each operand read once and each output written once; two operations per multiply-add (or per weight)."""
    nbytes = flops = 0
    m, group = case["m"], case["group"]
    for k, n in _shapes(case):
        nbytes += k * n // 2 + (k // group) * (2 * n + n // 2)
        if case["op"] == "dequant":
            nbytes += 2 * k * n
            flops += 2 * k * n
        else:
            nbytes += 2 * m * (k + n) + (4 * k if case["op"] != "gemm" else 0)
            flops += 2 * m * k * n
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Dequantised weights are exact by definition (one fp16 multiplication).  A product is rounded to fp16 once, and
    a kernel may contract the unrounded s * (q - z) or the weight rounded to fp16: against float64 the two differ by
    2e-4 and 3e-4 of the result, and by at most 1.6e-3 of the larger of the value and the result's size."""
    if case["op"] == "dequant":
        return "exact"
    return {"rel": 1.2e-3, "max": 6e-3}


def exact(case, seed):
    """The outputs in float64 from the definition, s * (q - z) with no rounding in between; a block of columns at a
    time, so that the widest layer fits beside the inputs."""
    state = prepare(dict(case, op="act_order" if case["op"] == "repacked" else case["op"], graph=False), seed)
    return [_exact(c, case["group"]) for c in state["calls"]]


def _exact(call, group):
    rows = call["qweight"].shape[0] * 8
    n = call["qweight"].shape[1]
    nibble = torch.arange(0, 32, 4, dtype=torch.int32, device="cuda")
    group_of = call.get("g_idx")
    if group_of is None:
        group_of = torch.arange(rows, device="cuda") // group
    group_of = group_of.long()
    x = call["x"].double() if "x" in call else None
    parts = []
    for lo in range(0, n, 8192):
        hi = min(n, lo + 8192)
        q = (call["qweight"][:, None, lo:hi] >> nibble[None, :, None] & 15).reshape(rows, hi - lo)
        z = (call["qzeros"][:, lo // 8:hi // 8, None] >> nibble & 15).reshape(-1, hi - lo)
        w = (q - z[group_of]).double().mul_(call["scales"][:, lo:hi].double()[group_of])
        parts.append(w if x is None else x @ w)
    return torch.cat(parts, dim=1)
