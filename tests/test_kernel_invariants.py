"""Properties of the compiled kernels that their speed or correctness counts on (no GPU needed).

1. What the 64-channel fp32 3x3 kernel's waits count on.

Without the add link the kernel issues the next tile's first two slab loads ahead of a tile's output stores and then
waits BY COUNT (vmcnt(45) / vmcnt(44): all but the other slab, the 32 stores and the 12 loads of the next patch).
That is only right if every wavefront really issues 32 stores and 12 patch loads per tile, whatever its lanes'
predicates: fewer operations after the slab than the wait allows to be outstanding and the slab may still be in
flight when it is read.  The compiler is free to branch around a store whose lanes are all off, to merge stores, or
to drop loads; this test fails the build of the library's sources if it ever does.

2. No wait for all vector-memory operations between two stores of an epilogue.  Every store of these epilogues sits
in a branch of its own; with a load still pending when such a branch is entered (a bias or addend value loaded inside
the epilogue) the compiler puts `s_waitcnt vmcnt(0)` in front of every store, and every store then waits for the one
before it to be written.  The kernels load those values ahead and state the wait once; this checks that it stays so.

3. Registers whose loads the compiler does not count are left alone until a wait has covered them, and the LDS that a kernel
addresses from zero starts there (what each is about stands with its test).
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_00907_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def _kernel_body(asm, mangled_piece):
    """Instructions and block labels of one kernel, in program text order."""
    m = re.search(r"^_ZN\S*" + mangled_piece + r"\S*:.*?\n(.*?)\.Lfunc_end", asm, re.S | re.M)
    assert m, mangled_piece
    lines = []
    for ln in m.group(1).splitlines():
        ln = ln.split(";")[0].strip()
        if ln and (ln.startswith(".LBB") or not ln.startswith(".")):
            lines.append(ln)
    return lines


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_k3c64_f32_issues_a_fixed_number_of_memory_operations_per_tile(tmp_path):
    out = tmp_path / "k3c64.s"
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-S", "--cuda-device-only",
           "-o", str(out), os.path.join(CSRC, "conv_k3c64_f32.hip")]
    subprocess.run(cmd, check=True, capture_output=True)
    body = _kernel_body(out.read_text(), "conv_k3c64_f32_kernelILb0E")       # the kernel without the add link
    stores = [i for i, ln in enumerate(body) if ln.startswith("buffer_store_dword")]
    assert len(stores) == 32, len(stores)                                    # one epilogue, 2 x 16 results per lane
    assert not any(ln.startswith(("global_store", "flat_store", "buffer_store_dwordx")) for ln in body)
    # nothing skips a store: a store under a lane predicate would sit between a branch on the exec mask and that
    # branch's (forward) target
    labels = {ln[:-1]: i for i, ln in enumerate(body) if ln.endswith(":")}
    for i, ln in enumerate(body):
        m = re.match(r"s_cbranch_exec(?:z|nz) (\S+)$", ln)
        if m and labels.get(m.group(1), -1) > i:
            skipped = [j for j in stores if i < j < labels[m.group(1)]]
            assert not skipped, (ln, len(skipped))
    # the patch fetch: twelve 16-byte loads at each of its two call sites (before the tile loop, inside it)
    patch_loads = [ln for ln in body if re.match(r"buffer_load_dwordx4 v\[", ln)]
    assert len(patch_loads) == 24, len(patch_loads)
    # the waits themselves: gfx9 encodes vmcnt in bits 3:0 and 15:14
    waits = set()
    for ln in body:
        m = re.match(r"s_waitcnt vmcnt\((\d+)\)$", ln)
        if m:
            waits.add(int(m.group(1)))
    assert {45, 44, 33, 32, 13, 12, 1, 0} <= waits, sorted(waits)


def _compile(tmp_path, name):
    out = tmp_path / (name + ".s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-S", "--cuda-device-only",
           "-o", str(out), os.path.join(CSRC, name + ".hip")]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text()


def _stores_that_wait(body):
    stores = [i for i, ln in enumerate(body) if re.match(r"(global|buffer|flat)_store", ln)]
    waits = 0
    for a, b in zip(stores, stores[1:]):
        if any(ln.startswith("s_waitcnt") and "vmcnt(0)" in ln for ln in body[a + 1:b]):
            waits += 1
    return len(stores), waits


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("source,kernel,n_stores", [
    ("conv_k3v_f32", "conv_k3v_f32_kernelILb0ELi7E", 112),          # 64 (squares) + 48 (strips of three blocks)
    ("conv_k3v_f32", "conv_k3v_f32_kernelILb0ELi8E", 128),
    ("igemm_f32_p3", "igemm_f32_p3_kernelILi2ELb0ELb0ELi3E", 32),
    ("igemm_f32_p3", "igemm_f32_p3_kernelILi2ELb1ELb1ELi3E", 32),
])
def test_no_epilogue_store_waits_for_the_one_before_it(tmp_path, source, kernel, n_stores):
    body = _kernel_body(_compile(tmp_path, source), kernel)
    stores, waiting = _stores_that_wait(body)
    assert stores == n_stores, stores
    assert waiting <= 2, waiting        # (the contraction over planes waits once per 32-channel column, by design)


def _registers(text):
    regs = set()
    for m in re.finditer(r"\bv(?:\[(\d+):(\d+)\]|(\d+))", text):
        regs.update(range(int(m.group(1)), int(m.group(2)) + 1) if m.group(1) else [int(m.group(3))])
    return frozenset(regs)


def _touched_in_flight(body, step):
    """Instructions that read or write a register whose load a wait has not yet covered, over every path through a kernel: (loads that
    were followed, such instructions).  Vector-memory operations finish in order; s_waitcnt vmcnt(n) leaves the last n.
    A step of the kernel's loop begins with the line `step`; a path on which a condition has left one out takes no further one (the
    conditions of the unrolled steps are those of a count that goes up)."""
    labels = {ln[:-1]: i for i, ln in enumerate(body) if ln.endswith(":")}
    todo, seen, loads, bad = [(0, (), False)], set(), set(), set()
    while todo:
        at, flying, left_out = todo.pop()
        while at < len(body):
            ln = body[at]
            if (at, flying, left_out) in seen or (left_out and ln == step):
                break
            seen.add((at, flying, left_out))
            op, _, rest = ln.partition(" ")
            if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
                to_register = "_load_" in op and not rest.split()[-1] == "lds"
                target = _registers(rest.split(",")[0]) if to_register else frozenset()
                if (_registers(rest) - target | target) & frozenset().union(*flying):
                    bad.add((at, ln))
                if target:
                    loads.add(at)
                flying = (flying + (target,))[-63:]
            elif op == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", rest)
                assert m or "lgkmcnt" in rest, ln
                if m:
                    flying = flying[len(flying) - min(len(flying), int(m.group(1))):]
            elif _registers(rest) & frozenset().union(*flying):
                bad.add((at, ln))
            if op == "s_endpgm":
                break
            m = re.match(r"s_(c?)branch\S* (\S+)$", ln)
            if m:
                if m.group(1):
                    to = labels[m.group(2)]
                    todo.append((to, flying, left_out or step in body[at:to] + body[at + 1:at + 4]))
                    left_out = left_out or step in body[to:to + 4]
                else:
                    at = labels[m.group(2)]
                    continue
            at += 1
    return loads, sorted(bad)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_registers_of_loads_in_assembly_are_left_alone_until_they_are_there(tmp_path):
    """fc_planes_f32.hip asks for the input's fragments in inline assembly, which the compiler does not count: a copy or spill of such a
    register between the load and the wait would take what was in it before.  Every path of both kernels is followed."""
    asm = _compile(tmp_path, "fc_planes_f32")
    for longk in (0, 1):
        body = _kernel_body(asm, f"igemm_f32_p3_fc_kernelILb{longk}E")
        loads, bad = _touched_in_flight(body, "s_waitcnt vmcnt(12)")
        assert not bad, bad[:5]
        assert loads == {i for i, ln in enumerate(body) if re.match(r"(buffer|global)_load", ln) and ln.split()[-1] != "lds"}, "every load is on some path"
        # what the check is worth: with the wait ahead of a slab's products gone (in the text alone), their operands are in flight
        waits = [i for i, ln in enumerate(body) if ln == "s_waitcnt vmcnt(12)"]
        assert len(waits) == 3, waits
        for w in waits:
            assert _touched_in_flight(body[:w] + ["s_nop 0"] + body[w + 1:], "s_waitcnt vmcnt(12)")[1]
    assert re.findall(r"\.(?:vgpr_spill_count|private_segment_fixed_size): +(\d+)", asm) == ["0"] * 4


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_the_block_kernels_dynamic_lds_starts_at_address_zero(tmp_path):
    """block_i8.hip's table of the addend's terms is addressed by the code alone: no LDS of a size known to the compiler may lie ahead of
    what the launch gives the kernel."""
    asm = _compile(tmp_path, "block_i8")
    sizes = re.findall(r"\.group_segment_fixed_size: +(\d+)", asm)
    assert sizes == ["0"] * 6, sizes


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("source,kernels", [("block_i8", 6), ("conv_dw", 12)])
def test_every_line_of_a_kernels_arguments_is_asked_for_at_its_start(tmp_path, source, kernels):
    """arguments.h: one load of each 64 bytes that the parameters lie in, whatever their number, ahead of the first wait."""
    asm = _compile(tmp_path, source)
    seen = 0
    for m in re.finditer(r"^  - \.agpr_count.*?\.name: +(\S+)$", asm, re.S | re.M):
        seen += 1
        ends = [int(o) + int(n) for o, n in re.findall(r"\.offset: +(\d+)\s+\.size: +(\d+)\s+\.value_kind: +(?:by_value|global_buffer)", m.group(0))]
        body = _kernel_body(asm, re.escape(m.group(1)[3:]))
        first = body[:next(i for i, ln in enumerate(body) if ln.startswith("s_waitcnt"))]
        got = {int(ln.rsplit(",", 1)[1], 16) for ln in first if ln.startswith("s_load_dword s")}
        assert got >= set(range(0, max(ends), 64)), (m.group(1), max(ends), sorted(got))
        assert max(got) < max(ends)
    assert seen == kernels, seen


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_two_workgroups_of_fc_few_f32_fit_a_compute_unit(tmp_path):
    """Sixteen wavefronts are four to a SIMD, whose 512 registers a lane hold eight of 64 each: with more than 256 tiles a kernel of 70 registers
    takes a second round."""
    asm = _compile(tmp_path, "fc_few_f32")
    counts = {}
    for block in re.split(r"\n  - \.a", asm):
        name, regs = re.search(r"\.name:\s+(\S+)", block), re.search(r"\.vgpr_count:\s+(\d+)", block)
        if name and regs and "fc_few_f32_kernel" in name.group(1):
            counts[name.group(1)] = int(regs.group(1)), int(re.search(r"\.vgpr_spill_count:\s+(\d+)", block).group(1))
    assert len(counts) == 7 and all(regs <= 64 and spilled == 0 for regs, spilled in counts.values()), counts
