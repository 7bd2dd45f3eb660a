"""Static checks over the compiled gfx950 ISA of the kernels that keep memory operations in flight behind the
compiler's back (CPU only: hipcc cross-compiles to assembly, nothing runs).

Two kernels issue loads as inline assembly and wait for them by hand, because the compiler's own counter
bookkeeping cost too much there: the mid-batch kernel (global loads of the weight stages, retired by one
`s_waitcnt vmcnt(n)` per stage) and the big-tile kernel (LDS reads of the A operands, retired by
`s_waitcnt lgkmcnt(n)`).  A third, the small-batch kernel on its ring, has its LDS slots refilled by DMA that the compiler
does not see.  The compiler does not know that the destination registers of such a load are still
pending: if it copied, reused or overwrote them between the load and the wait that retires it, a result would be
wrong only now and then.  Memory operations of one kind retire in order, so a walk along the paths of the code can tell.
"""
import os
import re
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2511_19438_amd import build as B

VM_PREFIXES = ("global_load", "global_store", "global_atomic", "buffer_", "scratch_", "flat_")


def compile_to_asm(src, defines, out_dir):
    out = os.path.join(out_dir, os.path.basename(src) + "".join(defines).replace("=", "_").replace("-D", ".") + ".s")
    cmd = [B.HIPCC, *B.COMMON, *defines, "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", out]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    assert proc.returncode == 0, proc.stderr[-2000:]
    return out


def kernels(path, labels=False):
    """{kernel name: instruction lines (directives and comments removed, labels too unless asked for; asm markers kept)}"""
    text = open(path).read()
    out = {}
    for m in re.finditer(r"^(_Z\w+):.*?\n(.*?)\.end_amdhsa_kernel", text, re.S | re.M):
        lines = []
        for raw in m.group(2).split("\n"):
            t = raw.strip()
            if t.startswith(";;#ASM"):
                lines.append(t)
                continue
            t = t.split(";")[0].strip()
            if t.endswith(":"):
                if labels:
                    lines.append(t)
                continue
            if not t or t.startswith("."):
                continue
            lines.append(t)
        out[m.group(1)] = lines
    return out


def vregs(operand):
    out = set()
    for m in re.finditer(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", operand):
        if m.group(1):
            out.update(range(int(m.group(1)), int(m.group(2)) + 1))
        else:
            out.add(int(m.group(3)))
    return out


def blocks(lines):
    """The basic blocks of a kernel's lines: [[(instruction, in inline assembly?)], [numbers of the blocks that may follow]]."""
    out, labels, in_asm = [[[], []]], {}, False
    for t in lines:
        if t.startswith(";;#ASM"):
            in_asm = t.startswith(";;#ASMSTART")
        elif t.endswith(":"):
            out.append([[], []])
            labels[t[:-1]] = len(out) - 1
        else:
            assert not t.startswith(("s_setpc", "s_swappc", "s_call", "s_cbranch_i_fork", "s_cbranch_g_fork")), t
            out[-1][0].append((t, in_asm))
            if t.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                out.append([[], []])
    for number, (code, successors) in enumerate(out):
        last = code[-1][0].split() if code else [""]
        if last[0].startswith(("s_branch", "s_cbranch")):
            successors.append(labels[last[1]])
        if last[0] not in ("s_branch", "s_endpgm") and number + 1 < len(out):
            successors.append(number + 1)
    return out


def walk(lines, step, without=()):
    """Follows every path through `lines` but those over the edges `without` (from one block to another).  What is in flight - {operation: how many behind it in the queue at least} - is
    handed to step(in_flight, instruction, in_asm), which changes it; where paths meet, an operation is in flight if it is on
    any of them, with the fewest behind it.  Step is called until nothing changes, and sees the weakest case of each place."""
    code = blocks(lines)
    entry = {0: {}}
    todo = [0]
    while todo:
        number = todo.pop()
        state = dict(entry[number])
        for t, in_asm in code[number][0]:
            step(state, t, in_asm)
        for nxt in code[number][1]:
            if (number, nxt) in without:
                continue
            known = entry.get(nxt)
            met = dict(state) if known is None else dict(known)
            if known is not None:
                for op, behind in state.items():
                    met[op] = min(behind, met.get(op, behind))
            if met != known:
                entry[nxt] = met
                if nxt not in todo:
                    todo.append(nxt)


def queue_up(state, op, counted=True):
    """`op` is issued; one that may overtake others (a scalar load) is no place in the queue for those before it."""
    if counted:
        for other in state:
            state[other] = min(state[other] + 1, 64)
    state[op] = 0


def retire(state, n):
    """A wait for at most n in flight: an operation with n or more behind it is done - one with fewer may not be."""
    for op in [op for op, behind in state.items() if behind >= n]:
        del state[op]


def check_pending(lines, is_tracked, is_counted, wait_re, what, without=()):
    """An instruction for which is_tracked(op, in_asm) holds puts its destination registers in flight; instructions for
    which is_counted(op) holds take a place in the in-order queue; `wait_re` extracts n from the waits.  No other
    instruction may name a register in flight, on any path."""
    problems = set()

    def step(state, t, in_asm):
        op = t.split()[0]
        if op == "s_waitcnt":
            m = wait_re.search(t)
            if m:
                retire(state, int(m.group(1)))
            return
        rest = t.partition(" ")[2]
        own, sources = frozenset(vregs(rest.split(",")[0])), vregs(rest.partition(",")[2])
        tracked = is_tracked(op, in_asm)
        for text, dest in state:
            # (a load of the same registers as a whole lands behind the one in flight: the queue is in order)
            if dest & sources or (dest & own and not (tracked and dest == own)):
                problems.add(f"{what}: '{t}' names v{sorted(dest & (own | sources))} while '{text}' is in flight")
        if is_counted(op):
            queue_up(state, (t, own if tracked else frozenset()), not op.startswith("s_"))

    walk(lines, step, without)
    return sorted(problems)


def check_refills(lines, what):
    """LDS reads that may still be on their way, on some path, when a DMA to LDS is issued."""
    problems = set()

    def step(state, t, in_asm):
        op = t.split()[0]
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", t)
            if m:
                retire(state, int(m.group(1)))
        elif op.startswith(("ds_", "s_load", "s_buffer_load")):
            queue_up(state, t, op.startswith("ds_"))
        elif re.match(r"(global|buffer)_load\w*_lds", op) or (op.startswith("buffer_load") and " lds" in t):
            problems.update(f"{what}: '{t}' while '{r}' is in flight" for r in state if r.startswith("ds_read"))

    walk(lines, step)
    return sorted(problems)


@pytest.fixture(scope="module")
def asm_files():
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    tmp = tempfile.mkdtemp(prefix="gptq_isa_")
    jobs = [("mid.hip", [])] + [("prefill_tile.hip", [f"-DGPTQ_PREFILL_TILE={t}"]) for t in B.PREFILL_TILES]
    jobs += [("ring.hip", [f"-DGPTQ_RING_GPU={g}"]) for g in B.RING_GROUPS]
    with ThreadPoolExecutor(max_workers=5) as pool:
        files = list(pool.map(lambda j: compile_to_asm(j[0], j[1], tmp), jobs))
    return {"mid": files[0], "prefill": files[1:1 + len(B.PREFILL_TILES)], "ring": files[1 + len(B.PREFILL_TILES):]}


def test_mid_batch_kernel_leaves_registers_of_pending_weight_loads_alone(asm_files):
    ks = {k: v for k, v in kernels(asm_files["mid"], labels=True).items() if "mid_kernel" in k}
    assert len(ks) >= 5
    wait = re.compile(r"vmcnt\((\d+)\)")
    for name, lines in ks.items():
        tracked = lambda op, in_asm: in_asm and op.startswith("global_load_dword")  # noqa: E731
        counted = lambda op: op.startswith(VM_PREFIXES)  # noqa: E731
        n_asm = sum(1 for i, t in enumerate(lines) if t.startswith("global_load_dword") and i and
                    lines[i - 1].startswith(";;#ASMSTART"))
        assert n_asm >= 18, f"{name}: expected the loop's weight loads as inline assembly, found {n_asm}"
        # Behind the loop stand the bodies of a first and of a second remaining stage: nobody runs the second without the first.
        code = blocks(lines)
        rest = [i for i, (block, _) in enumerate(code) if sum(in_asm and t.startswith("global_load_dword") for t, in_asm in block) == 6]
        assert len(rest) == 2, name
        first_left_out = {(i, n) for i, (_, nxt) in enumerate(code) if rest[0] in nxt for n in nxt if n != rest[0]}
        second_run = {(i, rest[1]) for i, (_, nxt) in enumerate(code) if rest[1] in nxt}
        assert first_left_out and second_run
        for without in (first_left_out, second_run):
            problems = check_pending(lines, tracked, counted, wait, name, without)
            assert not problems, "\n".join(problems[:10])


def test_big_tile_kernel_leaves_registers_of_pending_lds_reads_alone(asm_files):
    wait = re.compile(r"lgkmcnt\((\d+)\)")
    seen = 0
    for path in asm_files["prefill"]:
        for name, lines in kernels(path, labels=True).items():
            if "prefill_pipelined_kernel" not in name:
                continue
            seen += 1
            tracked = lambda op, in_asm: in_asm and op.startswith("ds_read")  # noqa: E731
            counted = lambda op: op.startswith("ds_") or op.startswith("s_load") or op.startswith("s_buffer_load")  # noqa: E731
            problems = check_pending(lines, tracked, counted, wait, name)
            assert not problems, "\n".join(problems[:10])
    assert seen >= 40


def check_mfma_wait_states(lines, what, valu_to_mfma=2, mfma_to_other=11):
    """MFMAs in inline assembly are unknown to the compiler's hazard checks: a vector instruction's result needs two wait
    states before an MFMA reads it, a sum of four passes eleven before anything but an MFMA touches it."""
    problems = []
    written, summed, now = {}, {}, 0
    for trip in range(2):
        for t in lines:
            if t.startswith(";;#"):
                continue
            op, _, rest = t.partition(" ")
            sums = {int(r) for m in re.finditer(r"\ba\[(\d+):(\d+)\]", rest) for r in range(int(m.group(1)), int(m.group(2)) + 1)}
            sums |= {int(m) for m in re.findall(r"\ba(\d+)\b", rest)}
            if op.startswith("v_mfma"):
                problems += [f"{what}: '{t}' {now - written[r]} after the write of v{r}"
                             for r in vregs(rest) if now - written.get(r, -99) <= valu_to_mfma]
                summed.update({r: now for r in sums})
            else:
                problems += [f"{what}: '{t}' {now - summed[r]} after the MFMA of a{r}"
                             for r in sums if now - summed.get(r, -99) <= mfma_to_other]
                if op.startswith("v_"):
                    written.update({r: now for r in vregs(rest.split(",")[0])})
            now += int(rest) + 1 if op == "s_nop" else 1
    return problems


def test_big_tile_kernel_leaves_wait_states_around_its_mfmas(asm_files):
    seen = 0
    for path in asm_files["prefill"]:
        for name, lines in kernels(path).items():
            if "prefill_pipelined_kernelILi256ELi256" in name:
                seen += 1
                assert sum(t.startswith("v_mfma") and " a[" in t for t in lines) >= 128
                problems = check_mfma_wait_states(lines, name)
                assert not problems, "\n".join(problems[:10])
    assert seen == 2


def test_the_wait_state_checker_flags_what_it_should():
    mfma = "v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], a[0:3]"
    assert check_mfma_wait_states(["v_perm_b32 v9, v1, v2, v3", "s_nop 1", mfma, "s_nop 15", "v_accvgpr_read_b32 v1, a2"], "good") == []
    assert len(check_mfma_wait_states(["v_perm_b32 v9, v1, v2, v3", mfma, "s_nop 15"], "early operand")) >= 1
    assert len(check_mfma_wait_states([mfma, "s_nop 3", "v_accvgpr_read_b32 v1, a2", "s_nop 15"], "early result")) >= 1


def test_ring_kernel_refills_a_slot_only_after_its_reads(asm_files):
    """A turn of the loop lets DMA into the slot that the turn before has read, scales and zero points included.  (None of
    its loads in inline assembly has a destination register: there are none in flight to leave alone.)"""
    seen = 0
    for path in asm_files["ring"]:
        for name, lines in kernels(path, labels=True).items():
            if "ring_kernel" not in name:
                continue
            seen += 1
            assert sum(t.startswith("global_load_lds") for t in lines) >= 6 and sum(t.startswith("ds_read") for t in lines) >= 8
            problems = check_refills(lines, name)
            assert not problems, "\n".join(problems[:10])
    assert seen >= 150


@pytest.mark.parametrize("files, kernel", [("ring", "ring_kernel"), ("prefill", "prefill_pipelined_kernel")])
def test_kernels_with_inline_dma_have_m0_to_themselves(asm_files, files, kernel):
    """The DMA's LDS address goes through m0, in inline assembly that cannot tell the compiler so: it may not use m0 itself."""
    for path in asm_files[files]:
        for name, lines in kernels(path).items():
            if kernel not in name:
                continue
            in_asm = False
            for t in lines:
                in_asm = t.startswith(";;#ASMSTART") or (in_asm and not t.startswith(";;#ASMEND"))
                assert in_asm or not re.search(r"\bm0\b", t), f"{name}: {t}"
            assert sum("m0" in t for t in lines) >= 6


def test_ring_kernels_registers_let_two_wavefronts_share_a_simd(asm_files):
    """Eight wavefronts of a workgroup, or two workgroups of four, as the plan's estimate takes it: 256 registers each, none spilled."""
    seen = 0
    for path in asm_files["ring"]:
        for entry in re.findall(r"^  - \.agpr_count:.*?(?=^  - |^amdhsa)", open(path).read(), re.S | re.M):
            if "ring_kernel" not in entry:
                continue
            seen += 1
            field = lambda name: int(re.search(rf"\.{name}:\s+(\d+)", entry).group(1))  # noqa: E731
            assert field("vgpr_count") <= 256 and field("vgpr_spill_count") == 0 and field("private_segment_fixed_size") == 0, entry
    assert seen >= 150


def test_the_refill_checker_flags_a_read_that_nothing_waits_for():
    loop = ["ds_read_b128 v[0:3], v8", "ds_read_b32 v4, v9", "s_waitcnt lgkmcnt(0)", "global_load_lds_dwordx4 v10, s[4:5]"]
    assert check_refills(loop, "good") == []
    assert len(check_refills(loop[:2] + ["s_waitcnt lgkmcnt(1)"] + loop[3:], "late")) >= 1
    assert len(check_refills(loop[:2] + loop[3:], "never")) >= 1


def test_the_checker_itself_flags_a_planted_violation():
    wait = re.compile(r"vmcnt\((\d+)\)")
    tracked = lambda op, in_asm: in_asm and op.startswith("global_load_dword")  # noqa: E731
    counted = lambda op: op.startswith(VM_PREFIXES)  # noqa: E731
    good = [";;#ASMSTART", "global_load_dwordx4 v[4:7], v1, s[2:3]", ";;#ASMEND",
            "global_load_lds_dwordx4 v2, s[4:5]",
            "v_add_u32 v8, v9, v10",
            ";;#ASMSTART", "s_waitcnt vmcnt(1)", ";;#ASMEND",
            "v_mov_b32 v11, v4",
            "s_waitcnt vmcnt(0)"]
    assert check_pending(good, tracked, counted, wait, "good") == []
    early_use = list(good)
    early_use[4] = "v_add_u32 v8, v5, v10"   # reads a register whose load has not been waited for
    assert len(check_pending(early_use, tracked, counted, wait, "early use")) >= 1
    clobber = list(good)
    clobber[4] = "v_mov_b32 v6, v10"          # hands a pending destination to something else
    assert len(check_pending(clobber, tracked, counted, wait, "clobber")) >= 1
    late_wait = list(good)
    late_wait[6] = "s_waitcnt vmcnt(2)"       # a wait that does not retire the load
    assert len(check_pending(late_wait, tracked, counted, wait, "late wait")) >= 1


def lds_problems(lines):
    return check_pending(lines, lambda op, in_asm: in_asm and op.startswith("ds_read"),
                         lambda op: op.startswith(("ds_", "s_load")), re.compile(r"lgkmcnt\((\d+)\)"), "planted")


def asm(text):
    return [";;#ASMSTART", text, ";;#ASMEND"]


def test_the_checker_flags_a_wait_for_more_reads_than_are_in_flight():
    """As many as the loop has in flight at this place, but fewer have been issued on the way into it: a wait for nothing."""
    reads = asm("ds_read_b128 v[0:3], v40") + asm("ds_read_b128 v[4:7], v40")
    use = ["v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[12:15], v[8:11]"]
    assert lds_problems(reads + asm("s_waitcnt lgkmcnt(1)") + use) == []
    for n in (2, 3, 12):
        assert lds_problems(reads + asm(f"s_waitcnt lgkmcnt({n})") + use) != [], n
    dma = "global_load_lds_dwordx4 v10, s[4:5]"
    assert check_refills(reads + ["s_waitcnt lgkmcnt(0)", dma], "good") == []
    assert check_refills(reads + ["s_waitcnt lgkmcnt(3)", dma], "none") != []


def test_the_checker_follows_branches():
    """A wait in a block that a path jumps over, a loop's next turn, and what only one of two ways leaves in flight."""
    read, use = asm("ds_read_b128 v[0:3], v40"), ["v_add_u32 v8, v1, v9"]
    skipped = read + ["s_cbranch_scc1 .LBB0_1", "s_waitcnt lgkmcnt(0)", ".LBB0_1:"] + use + ["s_endpgm"]
    assert lds_problems(skipped) != []
    assert lds_problems(read + ["s_branch .LBB0_1"] + use + [".LBB0_1:", "s_waitcnt lgkmcnt(0)"] + use + ["s_endpgm"]) == []
    loop = ["s_waitcnt lgkmcnt(0)", ".LBB0_1:"] + use + read + ["s_cbranch_scc1 .LBB0_1", "s_waitcnt lgkmcnt(0)", "s_endpgm"]
    assert lds_problems(loop) != []
    assert lds_problems(loop[:-3] + ["s_waitcnt lgkmcnt(0)"] + loop[-3:]) == []
    # the fewest reads behind the one in flight count, not those of the longer way
    joined = read + ["s_cbranch_scc1 .LBB0_1"] + asm("ds_read_b32 v20, v40") + [".LBB0_1:"] + asm("s_waitcnt lgkmcnt(1)") + use
    assert lds_problems(joined) != []
    # a scalar load may overtake the reads before it: it makes no place in the queue
    assert lds_problems(read + ["s_load_dword s4, s[0:1], 0x0"] + asm("s_waitcnt lgkmcnt(1)") + use) != []
