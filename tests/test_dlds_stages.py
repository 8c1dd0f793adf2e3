"""k_gemm_dlds in the built library: what its counted waits leave on their way.  A wave requests B's rows of K tile kt + 2, then A's of
kt + 3 (three stages of A; kt + 2 with two); a wait that leaves as many requests as A takes has all of B's and the older ones of A's."""
import re

import pytest

from test_lds_dma_waits import LANDED, VMEM, early_barriers, listings       # noqa: F401  (a fixture)


def scalars(operand):
    """Scalar registers that an operand names, and lanes of vector registers that hold one."""
    m = re.match(r"s(\d+)$|s\[(\d+):(\d+)\]$", operand)
    if m:
        return {"s%d" % r for r in ([int(m.group(1))] if m.group(1) else range(int(m.group(2)), int(m.group(3)) + 1))}
    return {operand} if operand in ("m0", "vcc_lo", "vcc_hi") else {"vcc_lo", "vcc_hi"} if operand == "vcc" else set()


def operands_of(code, region):
    """{index of a DMA: "A" or "B"}: B's go to LDS behind `region`, which enters their address as a constant.  Followed through the scalar
    instructions along every path; a DMA that is both on two paths is left out."""
    state, todo, found = {0: frozenset()}, [0], {}
    while todo:
        at = todo.pop()
        beyond = set(state[at])                           # registers with that constant in them
        op, text, target = code[at]
        args = [a.strip() for a in text.partition(" ")[2].split(",")]
        if text.endswith(" lds"):
            found.setdefault(at, set()).add("B" if "m0" in beyond else "A")
        elif op == "v_writelane_b32":
            cell = args[0] + "." + args[2]
            beyond = beyond | {cell} if scalars(args[1]) & beyond else beyond - {cell}
        elif op == "v_readlane_b32":
            beyond = beyond | scalars(args[0]) if args[1] + "." + args[2] in beyond else beyond - scalars(args[0])
        elif op.startswith(("s_", "v_readfirstlane")) and not op.startswith(("s_cmp", "s_waitcnt", "s_nop", "s_cbranch", "s_branch", "s_barrier", "s_endpgm", "s_bitcmp")):
            sources = set().union(*map(scalars, args[0 if op.startswith(("s_addk", "s_mulk", "s_cmov")) else 1:]))
            literal = op in ("s_add_i32", "s_add_u32", "s_addk_i32", "s_mov_b32") and any(re.match(r"0x[0-9a-f]+$", a) and int(a, 16) == region for a in args[1:])
            beyond = beyond | scalars(args[0]) if literal or sources & beyond else beyond - scalars(args[0])
        if op == "s_endpgm":
            continue
        for to in ([] if op == "s_branch" else [at + 1]) + ([] if target is None else [target]):
            was = state.get(to)
            now = frozenset(beyond) | (was or frozenset())
            if now != was:
                state[to] = now
                todo.append(to)
    return {at: min(kinds) for at, kinds in found.items() if len(kinds) == 1}


def early(code, operand, la):
    """Barriers that a wave may enter, along any path, with a request of B's on its way, or one of A's other than the `la` newest; program
    ends with any.  Kept of a path: the least number of operations behind B's requests, behind each of the `la` newest of A's, behind older ones."""
    state, todo, found = {0: (LANDED,) * (la + 2)}, [0], set()
    while todo:
        at = todo.pop()
        b, old, *new = state[at]
        op, text, target = code[at]
        if op.startswith(VMEM):
            b, old, new = min(b + 1, LANDED), min(old + 1, LANDED), [min(n + 1, LANDED) for n in new]
            if operand.get(at) == "B":
                b = 0
            elif text.endswith(" lds"):
                old, new = min(old, new[-1]), [0] + new[:-1]
        elif op == "s_waitcnt" and "vmcnt" in text:
            left = int(re.search(r"vmcnt\((\d+)\)", text).group(1))
            b, old, *new = [LANDED if n >= left else n for n in (b, old, *new)]
        elif op == "s_barrier" and min(b, old) < LANDED or op == "s_endpgm" and min(b, old, *new) < LANDED:
            found.add(at)
        if op == "s_endpgm":
            continue
        for to in ([] if op == "s_branch" else [at + 1]) + ([] if target is None else [target]):
            was = state.get(to, (LANDED + 1,) * (la + 2))
            now = tuple(map(min, was, (b, old, *new)))
            if now != was:
                state[to] = now
                todo.append(to)
    return found


def test_the_checks_themselves():
    dma, load, end = ("buffer_load_dwordx4", "buffer_load_dwordx4 v1, s[0:3], s4 offen lds", None), ("buffer_load_dword", "buffer_load_dword v9, v1, s[0:3], 0 offen", None), ("s_endpgm", "s_endpgm", None)
    wait, barrier, to = (lambda n: ("s_waitcnt", f"s_waitcnt vmcnt({n})", None)), ("s_barrier", "s_barrier", None), (lambda s: ("s_mov_b32", f"s_mov_b32 m0, {s}", None))
    add = ("s_add_i32", "s_add_i32 s8, s9, 0x18000", None)
    keep, back = ("v_writelane_b32", "v_writelane_b32 v3, s8, 5", None), ("v_readlane_b32", "v_readlane_b32 s7, v3, 5", None)
    assert operands_of([add, to("s8"), dma, to("s9"), dma, keep, back, to("s7"), dma, end], 0x18000) == {2: "B", 4: "A", 8: "B"}
    assert operands_of([add, ("s_mov_b32", "s_mov_b32 s8, 0", None), to("s8"), dma, end], 0x18000) == {3: "A"}
    good = [dma, dma, wait(1), barrier, wait(0), end]
    assert not early(good, {0: "B", 1: "A"}, 1) and early(good, {0: "A", 1: "B"}, 1) == {3}
    assert early([dma, dma, dma, wait(2), barrier, wait(0), end], {0: "B"}, 1) == {4}               # the older one of A's
    assert early([dma, dma, load, wait(2), barrier, wait(0), end], {0: "B"}, 1) == set() and early([dma, dma, load, wait(3), barrier, wait(0), end], {0: "B"}, 1) == {4}
    assert early([dma, wait(1), barrier, end], {}, 1) == {3}


@pytest.fixture(scope="module")
def forms(listings):                                       # noqa: F811
    found = []
    for name, code in listings.items():
        m = re.search(r"k_gemm_dldsILi(\d+)ELi(\d+)(?:ELi64)?ELi(\d+)ELi(\d+)E", name)
        if m:
            bm, bn, wr, wc = map(int, m.groups())
            found.append((name, code, bm, bn, wr * wc))
    assert found
    return found


def test_stages_have_landed_before_they_are_read(forms):
    three = 0
    for name, code, bm, bn, waves in forms:
        la, lb = bm // (8 * waves), bn // (8 * waves)
        if not (waves == 8 and (3 * bm + 2 * bn) * 128 <= 160 * 1024):
            assert not early_barriers(code, False), name   # two stages: every request has landed at the next barrier
            continue
        three += 1
        operand = operands_of(code, 3 * bm * 128)
        dmas = [at for at, (_, text, _) in enumerate(code) if text.endswith(" lds")]
        assert sorted(operand) == dmas and any(op == "s_barrier" for op, _, _ in code), name
        assert not early(code, operand, la), name
        waits = [int(n) for op, text, _ in code if op == "s_waitcnt" and "lgkmcnt(0)" in text for n in re.findall(r"vmcnt\((\d+)\)", text)]
        assert set(waits) <= {0, la} and waits.count(la) >= 3, (name, waits)
        loops = [(to, at) for at, (op, _, to) in enumerate(code) if to is not None and to < at]
        first, last = min((l for l in loops if sum(op.startswith("v_mfma") for op, _, _ in code[l[0]:l[1]])), key=lambda l: l[1] - l[0])
        vmem = [at for at in range(first, last) if code[at][0].startswith(("buffer_", "global_", "scratch_", "flat_"))]
        assert [operand.get(at) for at in vmem] == ["B"] * lb + ["A"] * la, (name, vmem)
        # with the loop's requests in the other order the check fails: the waits then leave B's on their way
        assert early(code, {**operand, **dict(zip(vmem, ["A"] * la + ["B"] * lb))}, la), name
    assert three
