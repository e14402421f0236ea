"""CPU test: what the compiler makes of the linear layers' kernels (assembly of gfx950, built here, nothing runs)."""
import os
import re
import subprocess

import pytest

from paper_2403_02310_amd import build


@pytest.fixture(scope="module")
def linear_assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "linear.s")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--offload-device-only", "-S", "-o", out,
                    os.path.join(build.CSRC, "linear_kernels.hip")], check=True, capture_output=True)
    return open(out).read()


WRITES_BEFORE, READS_AFTER = 2, 16   # wait states: what the instruction needs, and what the source puts behind the last one (it needs 8)


def registers(operand):
    """Registers of one operand: "v7", "a[0:3]"; nothing for scalars, literals and modifiers."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    first, last = (m[2], m[2]) if m[2] else (m[3], m[4])
    return {m[1] + str(r) for r in range(int(first), int(last) + 1)}


def instructions(body):
    """(opcode, operands, wait states, indices of what may run next) of a function's assembly."""
    lines, labels = [], {}
    for l in body.splitlines():
        l = l.split(";")[0].strip()
        if l.endswith(":"):
            labels[l[:-1]] = len(lines)
        elif l and not l.startswith("."):
            lines.append(l)
    out = []
    for i, l in enumerate(lines):
        op, _, rest = l.partition(" ")
        rest = rest.strip()
        if op.startswith("s_cbranch"):
            after = [i + 1, labels[rest]]
        elif op == "s_branch":
            after = [labels[rest]]
        else:
            after = [] if op == "s_endpgm" else [i + 1]
        out.append((op, [o for o in re.split(r",\s*", rest) if o], int(rest) + 1 if op == "s_nop" else 1, [a for a in after if a < len(lines)]))
    return out


def in_place_hazards(body):
    """Instructions too close to an in-place matrix instruction on any path: vector writes of its operands in front of it, and reads or
    writes of its result behind it, other matrix instructions on the same registers aside."""
    code = instructions(body)
    before = [[] for _ in code]
    for i, (_, _, _, after) in enumerate(code):
        for a in after:
            before[a].append(i)
    mfma = [i for i, (op, ops, _, _) in enumerate(code) if op == "v_mfma_f32_16x16x32_bf16" and ops[0].startswith("a") and ops[0] == ops[3]]
    found = []
    for i in mfma:
        result, operands = registers(code[i][1][0]), set().union(*(registers(o) for o in code[i][1]))
        reached, todo = {}, [(b, 0) for b in before[i]]
        while todo:   # wait states between the instruction and i
            j, states = todo.pop()
            if states >= WRITES_BEFORE or reached.get(j, WRITES_BEFORE) <= states:
                continue
            reached[j] = states
            op, ops, takes, _ = code[j]
            if op.startswith("v_") and "mfma" not in op and ops and registers(ops[0]) & operands:
                found.append((op, ops, "before", code[i][1]))
            todo += [(b, states + takes) for b in before[j]]
        reached, todo = {}, [(a, 0) for a in code[i][3]]
        while todo:
            j, states = todo.pop()
            if states >= READS_AFTER or reached.get(j, READS_AFTER) <= states:
                continue
            reached[j] = states
            op, ops, takes, after = code[j]
            same = "mfma" in op and ops[0] == code[i][1][0] and ops[3] == ops[0] and not any(registers(o) & result for o in ops[1:3])
            if not same and any(registers(o) & result for o in ops):
                found.append((op, ops, "after", code[i][1]))
            todo += [(a, states + takes) for a in after]
    return len(mfma), found


def phased_kernels(assembly):
    bodies = re.findall(r"^(\S*linear_phased_kernel\S*):.*?\n(.*?)^\.Lfunc_end", assembly, re.S | re.M)
    assert len(bodies) == 21
    return bodies


def test_in_place_matrix_instructions_keep_their_distances(linear_assembly):
    """The matrix instructions of the large tiles are inline assembly, which the compiler neither waits for nor keeps clear of; the sums are
    right only as long as no copy or spill comes near them."""
    for name, body in phased_kernels(linear_assembly):
        count, hazards = in_place_hazards(body)
        assert count >= 32 and not hazards, (name, hazards[:3])
        about = linear_assembly[linear_assembly.index(".name:           " + name):][:2000]
        assert re.search(r"\.private_segment_fixed_size: (\d+)", about)[1] == "0" and re.search(r"\.vgpr_spill_count: (\d+)", about)[1] == "0", name


@pytest.mark.parametrize("nops,line,where,caught", [
    (0, "v_accvgpr_read_b32 v1, {c}", 1, True), (15, "v_accvgpr_read_b32 v1, {c}", 1, True), (16, "v_accvgpr_read_b32 v1, {c}", 1, False),
    (0, "v_accvgpr_write_b32 {c}, 0", 1, True), (0, "scratch_store_dwordx4 off, {call}, off", 1, True), (0, "ds_write_b128 v1, {call}", 1, True),
    (0, "v_mov_b32_e32 {a}, v1", 0, True), (1, "v_mov_b32_e32 {a}, v1", 0, True), (2, "v_mov_b32_e32 {a}, v1", 0, False), (0, "v_accvgpr_mov_b32 {c}, a0", 0, True),
    (0, "s_mov_b32 s0, 0", 0, False), (0, "v_mov_b32_e32 v255, 0", 0, False),
])
def test_instructions_too_close_to_a_matrix_instruction_are_found(linear_assembly, nops, line, where, caught):
    """Planted in the text of the last matrix instruction of a kernel, which the sixteen wait states follow."""
    name, body = phased_kernels(linear_assembly)[0]
    lines = body.splitlines()
    at = max(i for i, l in enumerate(lines) if "v_mfma" in l)
    ops = [o.strip() for o in lines[at].split(None, 1)[1].split(",")]
    one = lambda o: sorted(registers(o))[0]  # noqa: E731
    planted = [line.format(c=one(ops[0]), call=ops[0], a=one(ops[1]))]
    wait = ["s_nop %d" % (min(nops, 8) - 1)] * (nops > 0) + ["s_nop %d" % (nops - 9)] * (nops > 8)
    new = lines[:at] + planted + wait + lines[at:] if where == 0 else lines[:at + 1] + wait + planted + lines[at + 1:]
    assert bool(in_place_hazards("\n".join(new))[1]) == caught


def test_output_strips_are_ordered_between_the_lanes_of_a_wavefront(linear_assembly):
    """The way out of a large tile turns 32 tokens at a time in LDS: lanes read what other lanes of the wavefront wrote.  The
    source states the order (a wavefront barrier, for which no instruction is issued) and the compiler keeps it: behind
    the key loop no LDS read follows LDS writes without one in between."""
    for name, body in phased_kernels(linear_assembly):
        lines = [l.strip() for l in body.splitlines()]
        start = max(i for i, l in enumerate(lines) if l.startswith("s_barrier"))
        written, reads = False, 0
        for l in lines[start:]:
            if "wave barrier" in l:
                written = False
            elif l.startswith("ds_write"):
                written = True
            elif l.startswith("ds_read"):
                assert not written, (name, l)
                reads += 1
        assert reads >= 12, name
