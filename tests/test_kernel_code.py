"""The compiled code of the product kernels.  The hand-ordered one: what inline assembly has requested into registers is not
touched before it is waited for, and the main loop holds nothing that keeps the matrix cores waiting.

The compiler takes the output of an inline-assembly load as written at once.  It may then copy,
spill or reuse the register while the data is still on its way (it does, where the K loop's body appears
twice).  So the LDS reads of the main loop are followed here through the control flow of every
instantiation, from the read to the wait behind it, and loads or returning atomics from global memory,
whose waits depend on how many copies are in flight, are not written as inline assembly at all.  The general
kernel's main loop waits for global memory once a slab."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2401_16677_amd import build as hip_build

SMALL = [u for u in hip_build.UNITS if u[0] == "t3_small_launch.hip" and "-DT3_MODE=1" in u[2]]
LAYOUTS = [u for u in hip_build.UNITS if u[0] == "t3_wide_launch.hip"]
GENERAL = [u for u in hip_build.UNITS if u[0] == "t3_gemm_launch.hip"]
API = [u for u in hip_build.UNITS if u[0] == "t3_api.hip"]


def _compile(out, units, kernel):
    """unit -> {kernel: lines} of the device assembly."""

    def compile_unit(unit):
        src, obj, defines = unit
        path = os.path.join(out, obj + ".asm")
        flags = [f for f in hip_build.HIPCC_FLAGS if f != "-Wall"]
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-w", *defines, "-I",
                        os.path.join(hip_build.ROOT, "include"), "-I", hip_build.CSRC, "--cuda-device-only", "-S",
                        os.path.join(hip_build.CSRC, src), "-o", path], check=True, stderr=subprocess.DEVNULL)
        with open(path) as f:
            text = f.read()
        starts = [m for m in re.finditer(r"^(_ZN\S+%s\S+):" % kernel, text, re.M)]
        return {m.group(1): text[m.end():text.index(".Lfunc_end", m.end())].split("\n") for m in starts}

    with ThreadPoolExecutor(4) as pool:
        return dict(zip([u[1] for u in units], pool.map(compile_unit, units)))


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    return _compile(tmp_path_factory.mktemp("asm"), LAYOUTS, "wide_tile_kernel")


@pytest.fixture(scope="module")
def general(tmp_path_factory):
    return _compile(tmp_path_factory.mktemp("asm"), GENERAL, "gemm_tile_kernel")


def _registers(text):
    """Vector registers an operand list names: v5, v[4:7], a3, a[0:3]."""
    regs = set()
    for kind, lo, hi, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))", text):
        if one:
            regs.add((kind, int(one)))
        else:
            regs.update((kind, i) for i in range(int(lo), int(hi) + 1))
    return regs


def _blocks(lines):
    """[(instructions, successors)], an instruction being (text, in inline assembly)."""
    blocks, labels, cur, asm = [], {}, [], False

    def close():
        nonlocal cur
        blocks.append(cur)
        cur = []

    for line in lines:
        label = re.match(r"^(\.LBB\w+):", line)
        if label:
            close()
            labels[label.group(1)] = len(blocks)
            continue
        if "#ASMSTART" in line or "#ASMEND" in line:
            asm = "#ASMSTART" in line
            continue
        text = line.split(";")[0].strip()
        if not text or text.startswith("."):
            continue
        cur.append((text, asm))
        if re.match(r"s_c?branch|s_endpgm", text):
            close()
    close()
    result = []
    for i, b in enumerate(blocks):
        succ, last = [], b[-1][0] if b else ""
        if last.startswith("s_branch"):
            succ = [labels[last.split()[1]]]
        elif last.startswith("s_cbranch"):
            succ = [labels[last.split()[1]], i + 1]
        elif not last.startswith("s_endpgm"):
            succ = [i + 1]
        result.append((b, [s for s in succ if s < len(blocks)]))
    return result


def _touched_in_flight(lines):
    """Instructions that name a register an inline-assembly LDS read may still be on its way to."""
    blocks = _blocks(lines)
    entry = [set() for _ in blocks]
    todo, faults, reads = list(range(len(blocks))), set(), 0
    while todo:
        i = todo.pop()
        pending = set(entry[i])
        for text, asm in blocks[i][0]:
            if text.startswith("s_waitcnt") and "lgkmcnt(0)" in text:
                pending.clear()
                continue
            op, _, rest = text.partition(" ")
            if _registers(rest) & pending:
                faults.add(text)
            if asm and op.startswith("ds_read"):
                pending |= _registers(rest.split(",")[0])
        for s in blocks[i][1]:
            if not pending <= entry[s]:
                entry[s] |= pending
                todo.append(s)
    reads = sum(asm and t.startswith("ds_read") for b, _ in blocks for t, asm in b)
    return faults, reads


def test_checker_sees_a_copy_of_a_register_in_flight():
    loop = [".LBB0_1:", "\t;;#ASMSTART", "\tds_read_b128 v[4:7], v0 offset:16", "\t;;#ASMEND", "{}",
            "\ts_cbranch_scc1 .LBB0_1", "\ts_waitcnt lgkmcnt(0)", "\tv_mov_b32_e32 v1, v4", "\ts_endpgm"]
    good = [line.format("\tv_mov_b32_e32 v1, v3") for line in loop]
    bad = [line.format("\tv_accvgpr_write_b32 a2, v6") for line in loop]
    # (a second pass through the loop asks for the same registers again: in the kernel a wait lies between)
    assert _touched_in_flight(good[:5] + good[6:])[0] == set()
    assert "v_accvgpr_write_b32 a2, v6" in _touched_in_flight(bad)[0]


@pytest.mark.parametrize("unit", [u[1] for u in LAYOUTS])
def test_no_register_in_flight_is_touched(code, unit):
    assert len(code[unit]) == 5                       # the five tiles
    for kernel, lines in code[unit].items():
        faults, reads = _touched_in_flight(lines)
        assert reads >= 24, kernel                    # (the smallest tile's two k-steps and the first one's)
        assert not faults, (kernel, sorted(faults)[:5])


@pytest.mark.parametrize("unit", [u[1] for u in LAYOUTS])
def test_no_global_load_to_a_register_in_inline_assembly(code, unit):
    for kernel, lines in code[unit].items():
        for block, _ in _blocks(lines):
            for text, asm in block:
                if asm and re.match(r"(global|buffer|flat|scratch)_(load|atomic)", text):
                    assert re.search(r"\blds\b", text) or text.split()[0].startswith("global_load_lds"), (kernel, text)


@pytest.mark.parametrize("unit", [u[1] for u in LAYOUTS])
def test_nothing_stands_between_the_products(code, unit):
    """One wavefront per SIMD: what the compiler puts between two products is time the matrix cores idle.
    No register is spilled to memory; where products are, the compiler waits for no memory access (its own
    accesses are on their way to registers the loop does not use); behind the barrier of a slab the first product
    follows at once, its addresses formed before."""
    for kernel, lines in code[unit].items():
        blocks = _blocks(lines)
        halves = 0
        for block, _ in blocks:
            assert not any(t.startswith("scratch_") for t, _ in block), kernel
            products = [i for i, (t, _) in enumerate(block) if t.startswith("v_mfma")]
            if len(products) < 8:
                continue
            assert not any(t.startswith("s_waitcnt") and "vmcnt" in t for t, asm in block if not asm), kernel
            if any(re.search(r"\blds\b", t) for t, _ in block):       # the half of a slab that copies: behind the barrier
                halves += 1
                assert products[0] <= 4, (kernel, block[:products[0]])
        assert halves == 1, kernel


@pytest.mark.parametrize("unit", [u[1] for u in LAYOUTS])
def test_argument_is_requested_once(code, unit):
    """The launch plan comes in two vector loads; the only scalar load is the tracker's generation.  Nothing goes through
    a pointer whose address space the compiler does not know."""
    for kernel, lines in code[unit].items():
        text = [t for block, _ in _blocks(lines) for t, _ in block]
        assert sum(t.startswith("global_load") for t in text) == 2, kernel
        assert sum(t.startswith("s_load") for t in text) <= 1, kernel
        assert not any(t.startswith("flat_") for t in text), kernel


@pytest.mark.parametrize("unit", [u[1] for u in GENERAL])
def test_general_main_loop_waits_once_a_slab(general, unit):
    """The loop over the slabs is one block that branches to itself.  Its copies stay in flight from one pass to the
    next: the only wait that names them is the one before the barrier, with the LDS accesses.  (A second one is what
    the compiler adds where an answer from memory, asked for behind an earlier branch, may still be on its way.)"""
    for kernel, lines in general[unit].items():
        loops = 0
        for i, (block, succ) in enumerate(_blocks(lines)):
            if i in succ and sum(t.startswith("v_mfma") for t, _ in block) >= 32:
                loops += 1
                waits = [t for t, _ in block if t.startswith("s_waitcnt") and "vmcnt" in t]
                assert len(waits) == 1 and "lgkmcnt(0)" in waits[0], (kernel, waits)
        assert loops == 1, kernel


def _waits_inside_a_batch(lines):
    """Whether a path leads from a load over a wait for global memory to another load, no store between."""
    blocks = _blocks(lines)
    seen, todo = set(), [(0, "none")]
    while todo:
        i, state = todo.pop()
        if (i, state) in seen:
            continue
        seen.add((i, state))
        for text, _ in blocks[i][0]:
            op = text.split()[0]
            if re.match(r"(global|flat)_load", op):
                if state == "waited":
                    return True
                state = "loaded"
            elif re.match(r"(global|flat)_store", op):
                state = "none"
            elif op == "s_waitcnt" and "vmcnt" in text and state == "loaded":
                state = "waited"
        todo += [(s, state) for s in blocks[i][1]]
    return False


def test_all_gather_step_requests_a_batch_at_once(tmp_path):
    """A lane's loads of a batch are all on their way before the first is waited for, but where fewer are
    meant to be."""
    (code,) = _compile(tmp_path, API, "ag_copy_kernel").values()
    assert len(code) == 9
    for kernel, lines in code.items():
        team, batch, in_flight = map(int, re.search(r"ILi(\d+)ELi(\d+)ELi(\d+)E", kernel).groups())
        assert sum(t.startswith("global_load") for b, _ in _blocks(lines) for t, _ in b) == batch, kernel
        assert _waits_inside_a_batch(lines) == (in_flight < batch), kernel
        # (nothing behind the call's own 48 bytes of arguments: a kernel that asks for the size of its grid has the host
        # write as many again with every launch)
        args = [int(m.group(1), 0) for line in lines for m in [re.match(r"\s*s_load_dword\S* \S+, s\[\d+:\d+\], (\w+)", line)] if m]
        assert args and max(args) < 48, (kernel, args)


@pytest.mark.parametrize("unit", [u[1] for u in SMALL])
def test_first_copies_do_not_wait_for_the_generation(unit, tmp_path):
    """The small-tile kernel: one scalar load that is not of the argument, the tracker's generation, and no wait for scalar loads
    between it and the first copies.  The instantiations that take the argument by vector have no other."""
    kernels = _compile(str(tmp_path), [u for u in SMALL if u[1] == unit], "small_tile_kernel")[unit]
    by_vector = 0
    for kernel, lines in kernels.items():
        text = [t for block, _ in _blocks(lines) for t, _ in block]
        loads = [i for i, t in enumerate(text) if t.startswith("s_load")]
        generation = [i for i in loads if ", s[0:1], " not in text[i]] or loads
        by_vector += len(loads) == 1
        copies = [i for i, t in enumerate(text) if t.startswith("global_load_lds")]
        assert len(generation) == 1 and generation[0] < copies[0], kernel
        assert not any(t.startswith("s_waitcnt") and "lgkmcnt" in t for t in text[generation[0]:copies[0]]), kernel
    assert by_vector == len(kernels) // 2
