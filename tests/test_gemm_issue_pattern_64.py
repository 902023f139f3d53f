"""The static check of test_gemm_issue_pattern.py for the 64-scene tile: between
two stage barriers each lane issues 4 library loads and one copy into LDS, nothing
else that counts against vmcnt, so that "at most 10 outstanding" means the stage
about to be used has landed."""
import re

from tests.test_gemm_issue_pattern import VMEM, asm, pytestmark  # noqa: F401

COPY = re.compile(r"buffer_load_dwordx4\b.*\blds\b")


def test_stage_issue_pattern_64(asm):  # noqa: F811
    names = re.findall(r"^(_ZN6psflib19gemm_h16_n64_kernel\w+):", asm, re.M)
    assert len(names) == 2  # bf16 and fp16
    for name in names:
        body = asm[asm.index(name + ":"):]
        lines = body[:body.index("s_endpgm")].splitlines()
        assert not any("scratch_" in l for l in lines), name
        bars = [i for i, l in enumerate(lines)
                if "s_barrier" in l and i > 0 and "s_waitcnt vmcnt(10)" in lines[i - 1]]
        assert len(bars) >= 8, name
        for a, b in zip(bars, bars[1:]):
            ops = [l for l in lines[a:b] if VMEM.match(l)]
            loads = sum("global_load_dwordx4" in l for l in ops)
            copies = sum(COPY.search(l) is not None for l in ops)
            assert (loads, copies, len(ops)) == (4, 1, 5), (name, a, ops)
        for i, l in enumerate(lines):
            if "Loop Header" in l:
                nxt = [b for b in bars if b > i]
                if nxt:
                    assert not any(VMEM.match(x) for x in lines[i:nxt[0]]), (name, i)
