"""Wait states between the matrix operations and the inline-assembly LDS adds of their results
(CPU only). The compiler puts the 12 wait states that a v_mfma_i32_32x32x32_i8 result needs in
front of its own reads, and none in front of an asm statement, so the dedispersion kernels wait
by an s_nop of their own. On every path of the compiled kernels from a matrix operation to an
asm statement that reads its result there must be such a wait: the distance must not rest on
how the instructions between happen to be scheduled."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2101_00941_amd import build

WAIT_STATES = 12

REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _regs(operand):
    """Bit mask of the vector registers that an operand names (accumulation registers from bit 512)."""
    bits = 0
    for kind, lo, hi, one in REG.findall(operand):
        a, b = (int(lo), int(hi)) if lo else (int(one), int(one))
        bits |= ((1 << (b - a + 1)) - 1) << (a + (512 if kind == "a" else 0))
    return bits


def _blocks(lines):
    """Basic blocks of a function: label -> (instructions, successors). An instruction is
    (text, whether an asm statement holds it)."""
    blocks, name, body, in_asm = {}, "entry", [], False
    order = []

    def close(successors):
        blocks[name] = (body, successors)
        order.append(name)

    for line in lines:
        if ";;#ASM" in line:
            in_asm = "ASMSTART" in line
            continue
        label = re.match(r"(\.LBB\w+):", line)
        if label:
            close([label.group(1)])
            name, body = label.group(1), []
            continue
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        body.append((text, in_asm))
        op = text.split()[0]
        if op.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_setpc")):
            fall = f"{name}+"
            close([t for t in text.split()[1:] if t.startswith(".LBB")] + ([fall] if op.startswith("s_cbranch") else []))
            name, body = fall, []
    close([])
    return blocks, order


def _unwaited(lines):
    """The asm instructions that read a matrix result without an asm wait before them, and the
    number of asm reads of matrix results that the analysis saw at all."""
    blocks, order = _blocks(lines)
    state = {b: 0 for b in order}     # registers that hold results not yet waited for, at entry
    results = 0                       # registers that any matrix operation writes
    for body, _ in blocks.values():
        for text, _ in body:
            if text.startswith("v_mfma"):
                results |= _regs(text.split(",")[0])
    bad, reads, work = set(), set(), list(order)
    while work:
        b = work.pop()
        body, successors = blocks[b]
        pending, nops = state[b], 0
        for i, (text, in_asm) in enumerate(body):
            op, _, rest = text.partition(" ")
            operands = rest.split(",")
            if op == "s_nop" and in_asm:
                nops += int(operands[0], 0) + 1
                if nops >= WAIT_STATES:
                    pending = 0
                continue
            nops = 0
            if op.startswith("v_mfma"):
                pending |= _regs(operands[0])
                continue
            writes = op.startswith("v_") or "load" in op or op.startswith("ds_read")
            if in_asm:
                read = 0
                for o in operands[1 if writes else 0:]:
                    read |= _regs(o)
                if op == "ds_add_u32" and _regs(operands[1]) & results:
                    reads.add((b, i))
                if read & pending:
                    bad.add((b, i, text))
            if writes:
                pending &= ~_regs(operands[0])
        for s in successors:
            if s in state and state[s] | pending != state[s]:
                state[s] |= pending
                work.append(s)
    return bad, len(reads)


@pytest.mark.parametrize("source", ["strip.hip", "dedisp.hip"])
def test_asm_reads_of_matrix_results_wait(source, tmp_path):
    if not os.path.exists(build.HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    out = tmp_path / "kernels.s"
    r = subprocess.run([build.HIPCC, *build.CFLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o",
                        str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    checked = 0
    for name, text in re.findall(r"; -- Begin function (\S+)\n(.*?); -- End function", out.read_text(), re.S):
        if "v_mfma" not in text:
            continue
        bad, reads = _unwaited(text.splitlines())
        assert reads > 0, name
        assert not bad, f"{name}: {len(bad)} reads without a wait, first {sorted(bad)[0]}"
        checked += 1
    assert checked >= 2


def test_the_analysis_follows_paths():
    """Made-up listings: a read behind a branch, behind a short wait, behind a whole one."""
    mfma = "v_mfma_i32_32x32x32_i8 v[16:31], v[8:11], v[4:7], v[16:31]"
    add = [";;#ASMSTART", "ds_add_u32 v0, v20", ";;#ASMEND"]

    def wait(n):
        return [";;#ASMSTART", f"s_nop {n}", ";;#ASMEND"]
    assert _unwaited([mfma, *add])[0]
    assert _unwaited([mfma, "s_cbranch_scc1 .LBB0_1", *wait(11), ".LBB0_1:", *add])[0]
    assert _unwaited([".LBB0_1:", *add, mfma, "s_cbranch_scc1 .LBB0_1", "s_endpgm"])[0]
    assert _unwaited([mfma, *wait(10), *add])[0]
    assert _unwaited([mfma, "s_nop 15", *add])[0]           # the compiler's own, for something else
    assert _unwaited([mfma, *wait(11), *add]) == (set(), 1)
    assert _unwaited([mfma, "v_mov_b32_e32 v20, v1", *add])[0] == set()
    assert _unwaited([mfma, *add, *wait(11)])[0]
