"""The bf16 attention kernel writes its MFMAs as inline assembly, for which the compiler inserts no wait
states: the distances it needs are looked up in the assembly built from the source (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2512_07090_amd import build

SRC = "attend_bf16.hip"
# Wait states (instructions, s_nop N counting N + 1) that nothing but an MFMA may come near a result; the
# compiler leaves 8 behind its own v_mfma_f32_16x16x32_bf16, and a VALU result 2 ahead of one that reads it.
RESULT, OPERAND = 16, 2


def _regs(token):
    m = re.match(r"^[-|]*v(?:\[(\d+):(\d+)\]|(\d+))", token)
    if not m:
        return set()
    return set(range(int(m[1]), int(m[2]) + 1)) if m[1] else {int(m[3])}


def _read_write(op, ops):
    regs = [_regs(o) for o in ops]
    every = set().union(*regs)
    if op.startswith(("global_store", "ds_write", "scratch_store", "buffer_store", "s_")):
        return every, set()
    written = regs[0] if regs else set()
    if "permlane" in op and "swap" in op:
        written = every
    return every, written


def _kernels(text):
    """name -> instructions (line, opcode, operands, inline asm) in program order"""
    out, name, inline = {}, None, False
    for no, line in enumerate(text.splitlines(), 1):
        inline = (inline or "#ASMSTART" in line) and "#ASMEND" not in line
        if re.match(r"^_Z\w+:", line):
            name = line.split(":")[0]
            out[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        m = re.match(r"^\s+([a-z]\w+)\s*(.*)$", line.split(";")[0])
        if name and m and not m[1].startswith("."):
            ops = [o.strip().split(" ")[0] for o in re.split(r",\s*(?![^\[]*\])", m[2].strip())] if m[2].strip() else []
            out[name].append((no, m[1], ops, inline))
    return out


def _states(op, ops):
    return 1 + (int(ops[0], 0) if op == "s_nop" else 0)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, *build.FILE_FLAGS[SRC], "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, SRC), "-o", out], check=True, capture_output=True)
    found = {k: v for k, v in _kernels(open(out).read()).items() if "attend_bf16_kernel" in k}
    assert len(found) == 3 and all(sum(i[1].startswith("v_mfma") and i[3] for i in v) > 150 for v in found.values())
    return found


def test_results_are_left_alone_until_they_are_written(kernels):
    for name, code in kernels.items():
        for at, (no, op, ops, inline) in enumerate(code):
            if not (op.startswith("v_mfma") and inline):
                continue
            result, states = _regs(ops[0]), 0
            for no2, op2, ops2, _ in code[at + 1:]:
                if states >= RESULT or op2 in ("s_endpgm", "s_branch"):
                    break
                if op2.startswith("v_mfma"):
                    # the next one may take it as its accumulator in place, not as an operand
                    assert not result & (_regs(ops2[1]) | _regs(ops2[2])), (name, no, no2)
                else:
                    assert not result & _read_write(op2, ops2)[0], (name, no, no2, op2, states)
                states += _states(op2, ops2)


def test_operands_are_written_before_they_are_read(kernels):
    for name, code in kernels.items():
        for at, (no, op, ops, inline) in enumerate(code):
            if not (op.startswith("v_mfma") and inline):
                continue
            reads, states = set().union(*[_regs(o) for o in ops[1:]]), 0
            for no2, op2, ops2, _ in reversed(code[:at]):
                if states >= OPERAND:
                    break
                if op2.startswith("v_") and not op2.startswith("v_mfma"):
                    assert not reads & _read_write(op2, ops2)[1], (name, no2, no, op2)
                states += _states(op2, ops2)
