"""The matrix instructions written in asm (gemm.hip, mfma_into) in the built library: until a result has arrived, nothing but a matrix
instruction that adds to the same registers touches them, and no vector instruction writes an input right in front.  For its own instructions
the compiler sees to that; of these it does not know."""
import os
import re
import subprocess

import pytest

from paper_2501_04012_amd import build
from test_lds_dma_waits import OBJDUMP, code_objects, parse

SETTLE = 11                                               # instructions issued behind a 16x16x32 before other units may use its sum
FRESH = 2                                                 # issued between a vector write and a matrix instruction that reads the register


def registers(text):
    """Vector registers that an instruction names."""
    found = set()
    for one, lo, hi in re.findall(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]", text):
        found.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return found


def touched_early(code, start):
    """The first instruction behind the matrix instruction at `start` that uses its sum too early."""
    sums = registers(code[start][1].split(",")[0])
    todo, seen = [(start + 1, SETTLE)], {}
    while todo:
        at, left = todo.pop()
        if left <= 0 or at >= len(code) or seen.get(at, 0) >= left:
            continue
        seen[at] = left
        op, text, target = code[at]
        if op == "s_endpgm":
            continue
        if op.startswith("v_mfma"):
            d, a, b, c = (registers(part) for part in text.partition(" ")[2].split(",")[:4])
            if sums & (a | b) or sums & (c | d) and not sums == c == d:
                return text
        elif sums & registers(text):
            return text
        left -= int(text.split()[1], 0) + 1 if op == "s_nop" else 1
        todo += [] if op == "s_branch" else [(at + 1, left)]
        todo += [] if target is None else [(target, left)]
    return None


def ways_in(code):
    """Instructions that may come right in front of each."""
    found = [[] for _ in code]
    for at, (op, _, target) in enumerate(code):
        if op not in ("s_branch", "s_endpgm") and at + 1 < len(code):
            found[at + 1].append(at)
        if target is not None:
            found[target].append(at)
    return found


def written_late(code, before, start):
    """A vector instruction too close in front of the matrix instruction at `start` that writes one of its inputs."""
    inputs = set().union(*(registers(part) for part in code[start][1].partition(" ")[2].split(",")[1:4]))
    todo, seen = [(at, FRESH) for at in before[start]], {}
    while todo:
        at, left = todo.pop()
        if left <= 0 or seen.get(at, 0) >= left:
            continue
        seen[at] = left
        op, text, _ = code[at]
        if op.startswith("v_") and not op.startswith("v_mfma") and inputs & registers(text.split(",")[0].partition(" ")[2]):
            return text
        left -= int(text.split()[1], 0) + 1 if op == "s_nop" else 1
        todo += [(p, left) for p in before[at]]
    return None


def test_the_check_itself():
    mfma, other, use = ("v_mfma_f32_16x16x32_bf16", "v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]", None), ("s_mov", "s_mov_b32 s0, s1", None), ("v_add", "v_add_f32 v4, v2, v5", None)
    assert touched_early([mfma] + [other] * 10 + [use], 0)
    assert not touched_early([mfma] + [other] * 11 + [use], 0)
    assert not touched_early([mfma, mfma, ("s_nop", "s_nop 15", None), use], 0)
    another = lambda text: ("v_mfma_f32_16x16x32_bf16", "v_mfma_f32_16x16x32_bf16 " + text, None)
    assert not touched_early([mfma, another("v[0:3], v[8:11], v[12:15], v[0:3]")], 0)
    assert touched_early([mfma, another("v[4:7], v[0:3], v[12:15], v[4:7]")], 0) and touched_early([mfma, another("v[4:7], v[8:11], v[2:5], v[4:7]")], 0)
    assert touched_early([mfma, another("v[2:5], v[8:11], v[12:15], v[2:5]")], 0) and touched_early([mfma, another("v[4:7], v[8:11], v[12:15], v[0:3]")], 0)
    assert touched_early([mfma, ("s_cbranch_scc0", "s_cbranch_scc0", 12)] + [other] * 9 + [("s_endpgm", "s_endpgm", None), use], 0)


def test_the_check_of_inputs_itself():
    mfma, other = ("v_mfma_f32_16x16x32_bf16", "v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]", None), ("s_mov", "s_mov_b32 s0, s1", None)
    late = lambda code: written_late(code, ways_in(code), code.index(mfma))
    for r in (0, 3, 8, 15):
        write = ("v_mov_b32", f"v_mov_b32 v{r}, v40", None)
        assert late([write, mfma]) and late([write, other, mfma]) and not late([write, other, other, mfma]) and not late([write, ("s_nop", "s_nop 1", None), mfma])
    assert not late([("v_mov_b32", "v_mov_b32 v4, v8", None), mfma])                       # reads an input, writes another register
    jump = [("s_branch", "s_branch 2", 2), ("s_endpgm", "s_endpgm", None), mfma, ("v_mov_b32", "v_mov_b32 v9, v40", None), ("s_cbranch_scc0", "s_cbranch_scc0 2", 2)]
    assert late(jump)                                      # around a loop


def test_sums_are_left_alone_until_they_are_there(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump beside hipcc")
    seen = 0
    for i, obj in enumerate(code_objects(build.LIB_PATH)):
        path = tmp_path / f"{i}.o"
        path.write_bytes(obj)
        if b"k_gemm_packed" not in obj:
            continue
        lines = {}
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout.splitlines():
            name = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if name:
                at = lines.setdefault(name.group(1), [])
            elif lines and line.startswith("\t") and "//" in line:
                at.append(line)
        for name, text in lines.items():
            if "k_gemm_dlds" not in name and "k_gemm_packed" not in name:
                continue
            code = parse(text)
            before = ways_in(code)
            for x, (op, _, _) in enumerate(code):
                if op == "v_mfma_f32_16x16x32_bf16":
                    seen += 1
                    assert touched_early(code, x) is None, (name, code[x][1], touched_early(code, x))
                    assert written_late(code, before, x) is None, (name, code[x][1], written_late(code, before, x))
    assert seen > 1000
