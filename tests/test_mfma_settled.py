"""Sums of the matrix instructions written in asm (gemm.hip, mfma_into) in the built library: until a result has arrived, nothing but
a matrix instruction touches its registers.  For its own instructions the compiler sees to that; of these it does not know."""
import os
import re
import subprocess

import pytest

from paper_2501_04012_amd import build
from test_lds_dma_waits import OBJDUMP, code_objects, parse

SETTLE = 11                                               # instructions issued behind a 16x16x32 before other units may use its sum


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
        if not op.startswith("v_mfma") and sums & registers(text):
            return text
        left -= int(text.split()[1], 0) + 1 if op == "s_nop" else 1
        todo += [] if op == "s_branch" else [(at + 1, left)]
        todo += [] if target is None else [(target, left)]
    return None


def test_the_check_itself():
    mfma, other, use = ("v_mfma_f32_16x16x32_bf16", "v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]", None), ("s_mov", "s_mov_b32 s0, s1", None), ("v_add", "v_add_f32 v4, v2, v5", None)
    assert touched_early([mfma] + [other] * 10 + [use], 0)
    assert not touched_early([mfma] + [other] * 11 + [use], 0)
    assert not touched_early([mfma, mfma, ("s_nop", "s_nop 15", None), use], 0)
    assert touched_early([mfma, ("s_cbranch_scc0", "s_cbranch_scc0", 12)] + [other] * 9 + [("s_endpgm", "s_endpgm", None), use], 0)


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
            for x, (op, _, _) in enumerate(code):
                if op == "v_mfma_f32_16x16x32_bf16":
                    seen += 1
                    assert touched_early(code, x) is None, (name, code[x][1], touched_early(code, x))
    assert seen > 1000
