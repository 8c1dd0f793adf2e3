"""Waits of the kernels that leave loads in flight across a barrier, read off the library's own machine code.

Data that a DMA brings to LDS is read behind a barrier that every wave enters after waiting for its own DMAs.  Where younger loads
may stay on their way, that wait is a count: a DMA has landed once at least so many vector memory operations were issued behind
it.  Nothing in the source fixes how many the compiler leaves there, so it is counted here, along every path of the control flow:
for each DMA the least number of operations behind it at each wait."""
import os
import re
import struct
import subprocess

import pytest

from paper_2501_04012_amd import build

OBJDUMP = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "llvm", "bin", "llvm-objdump")
LANDED = 1 << 20                                          # of a count: the DMA is known to have landed
VMEM = ("buffer_load", "buffer_store", "global_load", "global_store", "scratch_load", "scratch_store", "flat_")


def code_objects(path):
    """The gfx950 code objects bundled in a host library."""
    blob, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + length] and size:
                yield blob[at + off:at + off + size]
            p += 24 + length
        at = blob.find(magic, at + 1)


def parse(lines):
    """[(mnemonic, text, index of a branch's target or None)] of one function's listing."""
    rows, index = [], {}
    for line in lines:
        text, _, note = line.partition("//")
        address = int(note.split(":")[0], 16)
        target = re.search(r"<[^>]*\+0x([0-9a-f]+)>", note)
        index[address] = len(rows)
        rows.append((text.split()[0], text.strip(), address, int(target.group(1), 16) if target else 0))
    start = rows[0][2]
    return [(op, text, index[start + t] if "branch" in op else None) for op, text, _, t in rows]


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump beside hipcc")
    found = {}
    for i, obj in enumerate(code_objects(build.LIB_PATH)):
        path = tmp_path_factory.mktemp("co") / f"{i}.o"
        path.write_bytes(obj)
        if b"k_gemm_packed" not in obj:
            continue
        lines = None
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout.splitlines():
            name = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if name:
                lines = found.setdefault(name.group(1), [])
            elif lines is not None and line.startswith("\t") and "//" in line:
                lines.append(line)
    return {name: parse(lines) for name, lines in found.items() if lines}


def early_barriers(code, ahead):
    """Barriers (instruction index, first on its path) that a wave may enter before its DMAs have landed: those issued since the
    barrier before, or with `ahead` those issued before that one (all of them at a path's first barrier).  An end of the program
    counts as such a barrier for every DMA."""
    state, todo, early = {(0, True): (LANDED, LANDED)}, [(0, True)], set()
    while todo:
        at, first = todo.pop()
        new, old = state[at, first]                       # least number of operations behind the DMAs since the last barrier, and older ones
        op, text, target = code[at]
        following = first
        if op.startswith(VMEM):
            new, old = min(new + 1, LANDED), min(old + 1, LANDED)
            if text.endswith(" lds") or "_lds_" in op:
                new = 0
        elif op == "s_waitcnt" and "vmcnt" in text:
            left = int(re.search(r"vmcnt\((\d+)\)", text).group(1))
            new, old = LANDED if new >= left else new, LANDED if old >= left else old
        elif op == "s_barrier":
            if old < LANDED or (new < LANDED and (first or not ahead)):
                early.add((at, first))
            new, old, following = LANDED, min(new, old), False
        elif op == "s_endpgm":
            if min(new, old) < LANDED:
                early.add((at, first))
            continue
        for to in ([] if op == "s_branch" else [at + 1]) + ([] if target is None else [target]):
            was = state.get((to, following), (LANDED + 1, LANDED + 1))
            now = min(was[0], new), min(was[1], old)
            if now != was:
                state[to, following] = now
                todo.append((to, following))
    return early


def test_the_count_itself():
    load, dma, end = ("buffer_load_dwordx4", "v[0:3], v4, s[0:3], 0 offen", None), ("buffer_load_dwordx4", "v4, s[0:3], 0 offen lds", None), ("s_endpgm", "", None)
    wait, barrier = (lambda n: ("s_waitcnt", f"vmcnt({n})", None)), ("s_barrier", "", None)
    assert not early_barriers([dma, load, wait(1), barrier, end], False)
    assert early_barriers([dma, load, wait(2), barrier, end], False)
    assert early_barriers([load, dma, wait(1), barrier, end], False)
    assert early_barriers([dma, ("s_cbranch_scc0", "", 3), load, wait(1), barrier, end], False)      # a path without the load
    assert not early_barriers([dma, wait(0), barrier, dma, load, barrier, load, wait(2), barrier, wait(0), end], True)
    assert early_barriers([dma, wait(0), barrier, dma, load, barrier, load, wait(3), barrier, wait(0), end], True)
    assert early_barriers([dma, barrier, wait(0), end], True)                                        # nothing in front: all must have landed
    assert early_barriers([dma, end], False)


@pytest.mark.parametrize("kernel,ahead", [("k_gemm_packed", False), ("k_gemm_f32_parts", True)])
def test_tiles_have_landed_before_they_are_read(listings, kernel, ahead):
    """A K tile of k_gemm_packed has landed at the barrier after its request, the split weights of k_gemm_f32_parts, requested two
    slices ahead, at the second."""
    names = [n for n in listings if kernel in n]
    assert names
    for name in names:
        assert sum(op == "s_barrier" for op, _, _ in listings[name]) >= 2, name
        assert not early_barriers(listings[name], ahead), name


def test_no_slice_waits_for_more_than_it_reads(listings):
    """Both halves of the K loop of k_gemm_f32_parts leave two rounds of fetches and one of split weights on their way: a branch between
    two loads, or a way round the loop's second half, has the compiler wait for more."""
    seen = 0
    for name, code in listings.items():
        form = re.search(r"k_gemm_f32_partsILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi\d+ELb1E", name)
        if not form:
            continue
        bm, bn, wr, wc = map(int, form.groups())
        waves = wr * wc
        ahead = 2 * (bm * 4 // (waves * 64)) + -(-(bn * 96 // 1024) // waves)
        loops = [code[to:at] for at, (op, _, to) in enumerate(code) if to is not None and to < at]
        body = min((b for b in loops if sum(op == "s_barrier" for op, _, _ in b) == 2), key=len)
        counts = [int(n) for op, text, _ in body if op == "s_waitcnt" for n in re.findall(r"vmcnt\((\d+)\)", text)]
        assert counts and min(counts) >= ahead, (name, counts)
        seen += 1
    assert seen
