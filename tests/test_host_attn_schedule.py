"""The assembly of the attention kernels whose LDS reads are inline assembly (no GPU): those with 32 rows per wavefront and those with 16 rows per workgroup.

The compiler does not know when such a read's registers are written, nor, in the backward kernels of head dimension 128, that a matrix instruction in assembly is
one.  What the source keeps by its order and its waits is checked in what the compiler makes of it."""
import os
import re

import pytest

from paper_2504_06095_amd import build

KERNELS = ("attn_core_bwd_dkv_wide_kernel", "attn_core_bwd_dq_wide_kernel", "attn_core_bwd_both_wide_kernel")
VALU_TO_MATRIX = 2    # wait states from a vector instruction's result to a matrix instruction that reads it
MATRIX_TO_VALU = 8    # from a matrix instruction of four passes to a vector instruction that touches its result


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "attn.s")
    build._run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.HIP_FLAGS, "-S", "--offload-device-only", "-I", os.path.join(build.ROOT, "include"),
                "-I", build.CSRC, os.path.join(build.CSRC, "ntp_attn_core.hip"), "-o", out])
    return open(out).read().splitlines()


def _symbols(assembly, kernel):
    """Line numbers at which the instantiations of a kernel begin."""
    return [i for i, l in enumerate(assembly) if re.match(rf"_Z\w*\d{kernel}(I\w*)?E\w*:", l)]


def _code(assembly, start):
    """(instructions of the kernel at a line as (opcode, operand register sets, text), label -> index)"""
    code, labels = [], {}
    for line in assembly[start + 1:]:
        line = line.split(";")[0].strip()
        if line.startswith(".Lfunc_end"):
            return code, labels
        if re.fullmatch(r"\.\w+:", line):
            labels[line[:-1]] = len(code)
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" ")
            code.append((op, [_registers(p.strip().split(" ")[0]) for p in rest.split(",")], line))
    raise AssertionError(f"no end of the kernel at line {start}")


def _registers(operand):
    m = re.fullmatch(r"-?\|?([vas])(?:\[(\d+):(\d+)\]|(\d+))\|?", operand)
    if not m:
        return frozenset()
    lo, hi = (m[4], m[4]) if m[4] else (m[2], m[3])
    return frozenset((m[1], i) for i in range(int(lo), int(hi) + 1))


def _in_flight_faults(code, labels):
    """Instructions that touch the destination of an LDS or scalar read that may still be in flight.  State: destinations of the reads in
    flight, oldest first; where paths meet, the union, aligned at the youngest
    (the youngest 32: twice what a wait can leave)."""
    state, work, faults = {0: ()}, [0], {}
    while work:
        i = work.pop()
        q, (op, operands, text) = state[i], code[i]
        touched = frozenset().union(*operands)
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", text)
            q = q if not m else q[max(len(q) - int(m[1]), 0):]
        else:
            hit = touched & frozenset().union(*q) if q else frozenset()
            if hit:
                faults[i] = (text, sorted(hit))
            if op.startswith(("ds_", "s_load", "s_buffer_load")):
                q = (*q, operands[0] if not op.startswith("ds_write") else frozenset())
        after = [] if op == "s_endpgm" else [labels[text.split()[1]]] if op == "s_branch" else [i + 1]
        if op.startswith("s_cbranch"):
            after.append(labels[text.split()[1]])
        for j in after:
            old, n = state.get(j), max(len(state.get(j, ())), len(q))
            pad = lambda s: (frozenset(),) * (n - len(s)) + s  # noqa: E731
            new = (q if old is None else tuple(a | b for a, b in zip(pad(old), pad(q))))[-32:]
            if new != old:
                state[j] = new
                work.append(j)
    return faults


def _without_waits(code):
    return [c if c[0] != "s_waitcnt" else ("s_waitcnt", c[1], "s_waitcnt vmcnt(0)") for c in code]


def _distance_faults(code):
    """Pairs closer than the hardware asks for, in the order of the text (one wait state an instruction, four a matrix instruction)."""
    at, vector, matrix, faults = 0, {}, {}, []
    for op, operands, text in code:
        read = frozenset().union(*operands[1:]) if len(operands) > 1 else frozenset()
        if op.startswith("v_mfma"):
            faults += [(vector[r][1], text) for r in read if r in vector and at - vector[r][0] < VALU_TO_MATRIX]
            at += 4
            matrix.update({r: (at, text) for r in operands[0]})
            continue
        if op.startswith("v_"):
            faults += [(matrix[r][1], text) for r in read | operands[0] if r in matrix and at - matrix[r][0] < MATRIX_TO_VALU]
        at += int(text.split()[1]) + 1 if op == "s_nop" else 1
        if op.startswith("v_"):
            vector.update({r: (at, text) for r in operands[0]})
            for r in operands[0]:
                matrix.pop(r, None)
    return faults


@pytest.mark.parametrize("kernel", KERNELS)
def test_registers_are_left_alone_while_reads_are_in_flight(assembly, kernel):
    code, labels = _code(assembly, *_symbols(assembly, kernel))
    assert sum(op.startswith("v_mfma") for op, _, _ in code) >= 128 and sum(op.startswith("ds_read") for op, _, _ in code) >= 64
    assert not any("scratch_" in text for _, _, text in code)
    faults = _in_flight_faults(code, labels)
    assert not faults, list(faults.values())[:5]
    assert _in_flight_faults(_without_waits(code), labels)  # (the check sees a missing wait)


# paired and not; 16 rows per workgroup: both head dimensions, backward with and without the delta values formed in it (fewest LDS reads of them)
@pytest.mark.parametrize("kernel,instantiations,reads", [("attn_core_bwd_both64_dma_kernel", 2, 128), ("attn_core_fwd64_dma_kernel", 2, 48), ("attn_core_fwd_small_kernel", 2, 24),
                                                         ("attn_core_bwd_small_kernel", 4, 64)])
def test_registers_are_left_alone_where_the_matrix_instructions_are_the_compilers(assembly, kernel, instantiations, reads):
    starts = _symbols(assembly, kernel)
    assert len(starts) == instantiations
    for start in starts:
        code, labels = _code(assembly, start)
        assert sum(op.startswith("ds_read") for op, _, _ in code) >= reads and not any("scratch_" in text for _, _, text in code)
        assert not _in_flight_faults(code, labels), assembly[start]
        assert _in_flight_faults(_without_waits(code), labels)


@pytest.mark.parametrize("kernel", KERNELS)
def test_results_are_read_far_enough_behind_their_instructions(assembly, kernel):
    code, _ = _code(assembly, *_symbols(assembly, kernel))
    faults = _distance_faults(code)
    assert not faults, faults[:5]
    # (the check sees a vector instruction right before the matrix instruction that reads its result, and right behind one)
    i = next(i for i, c in enumerate(code) if c[0].startswith("v_mfma"))
    for at, operand in ((i, 1), (i + 1, 0)):
        assert _distance_faults([*code[:at], ("v_mov_b32", [code[i][1][operand], frozenset()], "planted"), *code[at:]])
