"""Wait states around the matrix instructions written as inline assembly, on the assembly that the
compiler makes of the library.

The compiler inserts wait states for its own matrix instructions; it does not look into inline assembly.
The sources keep the distances by fences and instruction order (tiles.hpp, mfma_vgpr), which says
nothing about copies that a register allocator may put in between: hence this check of what came out.
  * v_mfma_f32_32x32x16_bf16 takes 8 passes; until 12 wait states have gone by no other instruction may read
    or write its result, except a matrix instruction that goes on accumulating in the very same registers;
  * a vector instruction's result may be an operand of a matrix instruction after 2 wait states.
Every instruction counts as one wait state, s_nop n as n + 1, a further matrix instruction as the 8 passes
for which the pipe, which all of a wave's matrix instructions go through, is not free for it."""
import os
import re
import subprocess

import pytest

from paper_2605_06374_amd import build

RESULT_WAIT, OPERAND_WAIT, PASSES = 12, 2, 8


def registers(text):
    """Vector and accumulation registers named in an operand: {("v", 3), ...}."""
    out = set()
    for kind, lo, hi, single in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo, hi = (int(lo), int(hi)) if lo else (int(single), int(single))
        out.update((kind, r) for r in range(lo, hi + 1))
    return out


def parse(text):
    """[(opcode, [operands], is inline assembly)], {label: index}"""
    code, labels, inline = [], {}, False
    for line in text.splitlines():
        if "ASMSTART" in line or "ASMEND" in line:
            inline = "ASMSTART" in line
            continue
        line = line.split(";")[0].strip()
        m = re.match(r"([.\w$]+):$", line)
        if m:
            labels[m.group(1)] = len(code)
        elif line and not line.startswith("."):
            op, _, rest = line.partition(" ")
            code.append((op, [x.strip() for x in rest.split(",")] if rest else [], inline))
    return code, labels


def waits(ins):
    op, args, _ = ins
    return int(args[0], 0) + 1 if op == "s_nop" else PASSES if op.startswith("v_mfma") else 1


def within(code, labels, start, limit):
    """(index, wait states in between) of the instructions that can follow `start` within `limit` of them."""
    best, todo = {}, [(start + 1, 0)]
    while todo:
        i, gone = todo.pop()
        if i >= len(code) or gone >= limit or best.get(i, limit) <= gone:
            continue
        best[i] = gone
        op, args, _ = code[i]
        after = gone + waits(code[i])
        if op.startswith(("s_branch", "s_cbranch")):
            todo.append((labels[args[0]], after))
        if op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            todo.append((i + 1, after))
    return best.items()


def violations(text):
    code, labels = parse(text)
    bad, seen = [], 0
    for i, (op, args, inline) in enumerate(code):
        if inline and op.startswith("v_mfma"):
            seen += 1
            result = registers(args[0])
            for j, gone in within(code, labels, i, RESULT_WAIT):
                op2, args2, _ = code[j]
                if op2.startswith("v_mfma"):
                    goes_on = args2[0] == args2[3] == args[0]
                    touched = args2[1:3] if goes_on else args2
                else:
                    touched = args2
                if any(registers(a) & result for a in touched):
                    bad.append(f"result of {i}: {op} {', '.join(args)} touched {gone} wait states later: {op2} {', '.join(args2)}")
        elif op.startswith("v_") and not op.startswith("v_mfma") and args:
            written = registers(args[0]) | (registers(args[1]) if "swap" in op else set())
            for j, gone in within(code, labels, i, OPERAND_WAIT):
                op2, args2, inline2 = code[j]
                if inline2 and op2.startswith("v_mfma") and any(registers(a) & written for a in args2[1:]):
                    bad.append(f"{op} {', '.join(args)} {gone} wait states before {op2} {', '.join(args2)}")
    return bad, seen


CHAIN = """
	;;#ASMSTART
	v_mfma_f32_32x32x16_bf16 v[0:15], v[32:35], v[36:39], 0
	;;#ASMEND
	;;#ASMSTART
	v_mfma_f32_32x32x16_bf16 v[0:15], v[40:43], v[44:47], v[0:15]
	;;#ASMEND
"""


@pytest.mark.parametrize("tail,count", [
    ("s_nop 15\nv_mul_f32 v16, v17, v3", 0),
    ("s_nop 10\nv_mul_f32 v16, v17, v3", 1),                     # read too early
    ("s_nop 10\nv_mov_b32 v3, 0", 1),                            # overwritten too early
    ("v_mfma_f32_32x32x16_bf16 a[0:15], v[48:51], v[52:55], a[0:15]\ns_nop 3\nv_exp_f32 v3, v3", 0),
    ("v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[52:55], a[0:15]", 2),   # an operand too early (the 9 and the 1 wait states behind both of the chain)
    ("s_cbranch_scc1 .L1\ns_nop 15\ns_endpgm\n.L1:\nds_write_b128 v20, v[0:3]", 2),
    ("v_mov_b32 v60, 0\n;;#ASMSTART\nv_mfma_f32_32x32x16_bf16 v[64:79], v[60:63], v[44:47], 0\n;;#ASMEND", 1),
    ("v_mov_b32 v60, 0\ns_nop 1\n;;#ASMSTART\nv_mfma_f32_32x32x16_bf16 v[64:79], v[60:63], v[44:47], 0\n;;#ASMEND", 0)])
def test_snippets(tail, count):
    bad, _ = violations(CHAIN + tail)
    assert len(bad) == count, bad


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the HIP compiler")
def test_inline_matrix_instructions_keep_their_distances(tmp_path):
    out = tmp_path / "varlen_attn.s"
    flags = [f for f in build.FLAGS if f != "-shared"]
    subprocess.run([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-o", str(out), build.SRC], check=True,
                   capture_output=True)
    bad, seen = violations(out.read_text())
    assert seen >= 100          # the check found what it is for
    assert not bad, "\n".join(bad[:20])


def transcendental_violations(text):
    """Exponentials written as inline assembly whose result a plain vector instruction takes in the very next wait state (one is needed)."""
    code, labels = parse(text)
    bad, seen = [], 0
    for i, (op, args, inline) in enumerate(code):
        if inline and op.startswith("v_exp"):
            seen += 1
            for j, _ in within(code, labels, i, 1):
                op2, args2, _ = code[j]
                if op2.startswith("v_") and not op2.startswith("v_mfma") and any(registers(a) & registers(args[0]) for a in args2):
                    bad.append(f"{op} {', '.join(args)} in front of {op2} {', '.join(args2)}")
    return bad, seen


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the HIP compiler")
def test_inline_exponentials_keep_their_distance(tmp_path):
    planted = ";;#ASMSTART\nv_exp_f32 v3, v4\n;;#ASMEND\n"
    assert [len(transcendental_violations(planted + t)[0]) for t in ("v_add_f32 v5, v3, v6", "s_nop 0\nv_add_f32 v5, v3, v6", "v_add_f32 v5, v7, v6")] == [1, 0, 0]
    out = tmp_path / "varlen_attn.s"
    flags = [f for f in build.FLAGS if f != "-shared"]
    subprocess.run([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-o", str(out), build.SRC], check=True, capture_output=True)
    bad, seen = transcendental_violations(out.read_text())
    assert seen >= 64
    assert not bad, "\n".join(bad[:20])


def load_violations(text):
    """Loads whose scalar operands are too fresh, none of which the compiler sees inside inline assembly: a load to LDS takes its destination from
    m0 one wait state behind a scalar write of it at the earliest, and an address in scalar registers five behind the vector instruction that wrote them."""
    scalars = lambda text: {r for lo, hi, one in re.findall(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)", text)
                            for r in (range(int(lo), int(hi) + 1) if lo else [int(one)])}
    code, labels = parse(text)
    bad, seen = [], 0
    for i, (op, args, _) in enumerate(code):
        if op.startswith("s_") and args and args[0] == "m0":
            seen += 1
            bad += [f"{op} {', '.join(args)} right in front of {code[j][0]}" for j, _ in within(code, labels, i, 1)
                    if "_lds_" in code[j][0] and code[j][0].startswith(("global_", "buffer_", "scratch_"))]
        elif op.startswith("v_") and args and scalars(args[0]):
            bad += [f"{op} {', '.join(args)} {gone} wait states before {code[j][0]} {', '.join(code[j][1])}"
                    for j, gone in within(code, labels, i, 5)
                    if code[j][0].startswith(("global_", "buffer_", "scratch_", "flat_")) and any(scalars(a) & scalars(args[0]) for a in code[j][1])]
    return bad, seen


@pytest.mark.parametrize("between,count", [("", 1), ("s_nop 0\n", 0), ("s_add_u32 s0, s0, s1\n", 0), ("s_branch .L1\n.L1:\n", 0),
                                           ("v_readfirstlane_b32 s5, v9\ns_nop 3\n", 1), ("v_readfirstlane_b32 s5, v9\ns_nop 4\n", 0)])
def test_load_snippets(between, count):
    planted = "s_add_u32 m0, s2, 64\n" + between + ";;#ASMSTART\nglobal_load_lds_dwordx4 v1, s[4:5] offset:64\n;;#ASMEND\n"
    assert len(load_violations(planted)[0]) == count


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs the HIP compiler")
def test_inline_loads_keep_their_distances(tmp_path):
    out = tmp_path / "varlen_attn.s"
    flags = [f for f in build.FLAGS if f != "-shared"]
    subprocess.run([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-o", str(out), build.SRC], check=True, capture_output=True)
    bad, seen = load_violations(out.read_text())
    assert seen >= 100
    assert not bad, "\n".join(bad[:20])
