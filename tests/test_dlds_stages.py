"""k_gemm_dlds in the built library: what its counted waits leave on their way.  A wave requests B's rows of K tile kt + 2, then A's of
kt + 3 (three stages of A; kt + 2 with two); a wait that leaves as many requests as A takes has all of B's and the older ones of A's."""
import re

from test_lds_dma_waits import early_barriers, listings       # noqa: F401  (a fixture)


def test_stages_have_landed_before_they_are_read(listings):    # noqa: F811
    names = [n for n in listings if "k_gemm_dlds" in n]
    assert names
    for name in names:
        bm, bn, wr, wc = map(int, re.search(r"k_gemm_dldsILi(\d+)ELi(\d+)ELi64ELi(\d+)ELi(\d+)E", name).groups())
        la, lb = bm // (8 * wr * wc), bn // (8 * wr * wc)
        three = wr * wc == 8 and (3 * bm + 2 * bn) * 128 <= 160 * 1024
        code = listings[name]
        early = early_barriers(code, three)
        # two stages: every request has landed at the next barrier; three: none is on its way when the program ends
        assert all(code[at][0] == "s_barrier" for at, _ in early) if three else not early, name
        if not three:
            continue
        waits = [int(n) for op, text, _ in code if op == "s_waitcnt" and "lgkmcnt(0)" in text for n in re.findall(r"vmcnt\((\d+)\)", text)]
        assert set(waits) <= {0, la} and waits.count(la) >= 3, (name, waits)
        loops = [code[to:at] for at, (op, _, to) in enumerate(code) if to is not None and to < at]
        body = min((b for b in loops if sum(op.startswith("v_mfma") for op, _, _ in b)), key=len)
        vmem = [text for op, text, _ in body if op.startswith(("buffer_", "global_", "scratch_", "flat_"))]
        assert len(vmem) == la + lb and all(t.endswith(" lds") for t in vmem), (name, vmem)
