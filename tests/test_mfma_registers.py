"""Registers of the matrix instructions in the built library: a sum lies in the registers of the sum it is added to, or in none of them.
Left to itself the compiler gives four-register sums outputs that overlap their input by two registers.  A build with such instructions
in its loops gave wrong sums; that they were the reason is inferred (the build without them differs in schedule and waits too)."""
import os
import re
import subprocess

import pytest

from paper_2501_04012_amd import build
from test_lds_dma_waits import OBJDUMP, code_objects


def partly_shared(text):
    """Whether the output of a matrix instruction overlaps its third input without being the same registers."""
    ops = [re.match(r"([va])\[(\d+):(\d+)\]$", o.strip()) for o in text.split(None, 1)[1].split(",")[:4]]
    if not ops[0] or not ops[3] or ops[0].group(1) != ops[3].group(1):
        return False
    (d0, d1), (c0, c1) = ((int(o.group(2)), int(o.group(3))) for o in (ops[0], ops[3]))
    return (d0, d1) != (c0, c1) and d0 <= c1 and c0 <= d1


def test_the_check_itself():
    assert not partly_shared("v_mfma_f32_16x16x4_f32 v[0:3], v8, v9, v[0:3]")
    assert not partly_shared("v_mfma_f32_16x16x4_f32 v[0:3], v8, v9, v[4:7]")
    assert not partly_shared("v_mfma_f32_16x16x4_f32 v[0:3], v8, v9, 0")
    assert not partly_shared("v_mfma_f32_16x16x4_f32 a[0:3], v8, v9, v[2:5]")
    assert partly_shared("v_mfma_f32_16x16x4_f32 v[0:3], v8, v9, v[2:5]")
    assert partly_shared("v_mfma_f32_32x32x16_bf16 v[16:31], v[0:3], v[4:7], v[4:19]")


def test_no_sum_shares_part_of_its_registers(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump beside hipcc")
    seen = 0
    for i, obj in enumerate(code_objects(build.LIB_PATH)):
        path = tmp_path / f"{i}.o"
        path.write_bytes(obj)
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout
        for line in out.splitlines():
            text = line.partition("//")[0].strip()
            if text.startswith("v_mfma"):
                seen += 1
                assert not partly_shared(text), text
    assert seen > 1000
