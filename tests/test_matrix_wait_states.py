"""Wait states round the matrix instructions that stand in inline assembly. The compiler puts them in for instructions that it knows
as such; it does not look into inline assembly, and nothing at run time shows a missing one for sure. So the assembly of the file is
read: along every path behind such an instruction, its result is neither read nor written by another kind of instruction for as long
as it is on its way, and no operand of it is written by a vector instruction right in front. No GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2303_04769_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
RESULT = 11          # wait states from an instruction of eight passes (16x16x32 bf16, 16x16x4 fp32) to another kind's use of its result
SOURCES = {"conv_split3_wide.hip": 864, "dwpw.hip": 350}          # and how many such instructions there are at least
OPERAND = 2          # from a vector instruction's result to a matrix instruction that reads it


def _regs(op):
    op = op.strip().strip("|-")
    m = re.match(r"([av])\[(\d+):(\d+)\]$", op)
    if m:
        return {(m[1], k) for k in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([av])(\d+)$", op)
    return {(m[1], int(m[2]))} if m else set()


def _program(text):
    """([(opcode, operand register sets, whether inside inline assembly, label of a branch)], label -> index)"""
    ins, labels, inside = [], {}, False
    for line in text.split("\n"):
        inside = ("#ASMSTART" in line) or (inside and "#ASMEND" not in line)
        code = line.split(";")[0].strip()
        if re.match(r"[.\w$]+:$", code):
            labels[code[:-1]] = len(ins)
        elif code and not code.startswith("."):
            op, _, rest = code.partition(" ")
            args = [a.strip() for a in rest.split(",")] if rest else []
            ins.append((op, [_regs(a) for a in args], inside, args[0] if op.startswith(("s_branch", "s_cbranch", "s_nop")) else None))
    return ins, labels


def _behind(ins, labels, k, limit):
    """(wait states passed, index) of the instructions that can follow instruction k within `limit`."""
    seen, todo = {}, [(k + 1, 0)]
    while todo:
        i, ws = todo.pop()
        if i >= len(ins) or ws >= limit or seen.get(i, limit) <= ws:
            continue
        seen[i] = ws
        op, _, _, arg = ins[i]
        yield ws, i
        if op == "s_endpgm":
            continue
        nxt = ws + (int(arg, 0) + 1 if op == "s_nop" else 1)
        if op.startswith(("s_branch", "s_cbranch")):
            todo.append((labels[arg], nxt))
        if op != "s_branch":
            todo.append((i + 1, nxt))


def faults(text):
    """Of a kernel's tied sums all count as the last one: in which order they are read is the compiler's choice."""
    ins, labels = _program(text)
    out, n = [], 0
    first = 0
    for end in [i + 1 for i, x in enumerate(ins) if x[0] == "s_endpgm"]:      # (a kernel may have several ends)
        tied = [i for i in range(first, end) if ins[i][0].startswith("v_mfma") and ins[i][2]]
        n += len(tied)
        sums = set().union(*[ins[i][1][0] for i in tied])
        for k in tied:
            for ws, i in _behind(ins, labels, k, RESULT):
                op, args, inside, _ = ins[i]
                # (of one kind: the chain of a sum, which the hardware waits for)
                if not (op.startswith("v_mfma") and inside) and any(sums & a for a in args):
                    out.append(f"result of instruction {k} met by {op} ({i}) after {ws}")
        first = end
    for k, (op, args, _, _) in enumerate(ins):
        if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp", "v_readfirstlane", "v_readlane")) and args:
            for ws, i in _behind(ins, labels, k, OPERAND):
                if ins[i][0].startswith("v_mfma") and ins[i][2] and any(args[0] & a for a in ins[i][1][1:]):
                    out.append(f"{op} ({k}) writes an operand of instruction {i}, {ws} behind it")
    return n, out


def test_the_reading():
    head = ";;#ASMSTART\nv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n;;#ASMEND\n"
    assert faults(head + "s_nop 10\nv_accvgpr_read_b32 v9, a2\ns_endpgm") == (1, [])
    for early in ("s_nop 9\nv_accvgpr_read_b32 v9, a2\n", "v_accvgpr_write_b32 a3, v1\n", "s_cbranch_scc1 L\ns_endpgm\nL:\nv_add_f32 v1, v2, a0\n"):
        assert len(faults(head + early + "s_endpgm")[1]) == 1, early
    assert len(faults("v_mov_b32 v5, 0\ns_nop 0\n" + head + "s_endpgm")[1]) == 1
    assert faults("v_mov_b32 v5, 0\ns_nop 1\n" + head + "s_endpgm") == (1, [])


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs the compiler")
@pytest.mark.parametrize("source,number", sorted(SOURCES.items()))
def test_wait_states(source, number, tmp_path):
    out = str(tmp_path / "a.s")
    flags = [f for f in build.FLAGS if f not in ("-Wall",)]
    subprocess.run([HIPCC] + flags + ["-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", out], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    n, found = faults(open(out).read())
    assert n >= number and not found, found[:5]


def test_every_file_with_such_instructions_is_read():
    files = [f for f in os.listdir(build.CSRC) if re.search(r'asm[^;]*"v_mfma', open(os.path.join(build.CSRC, f)).read())]
    assert sorted(files) == sorted(SOURCES)
