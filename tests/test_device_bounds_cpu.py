"""Rules of the device code that no run can show to be broken without risking a fault, checked
on the source: waits before asynchronous writes, indices clamped to their tables."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_23728_amd", "csrc")


def code(name):
    text = open(os.path.join(CSRC, name)).read()
    return re.sub(r"//[^\n]*", "", re.sub(r"/\*.*?\*/", "", text, flags=re.S))


def body(text, start):
    """The braced block that opens at or after `start`."""
    i = text.index("{", start)
    depth = 0
    for j in range(i, len(text)):
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        if depth == 0:
            return text[i:j + 1]
    raise AssertionError("unbalanced braces")


def test_asynchronous_lds_loads_wait_for_the_reads_before_them():
    """A load that writes LDS by the memory pipe is not ordered against LDS reads under way:
    the function that issues it waits for them (lgkmcnt) before its first one."""
    found = 0
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".h")) or "__builtin_amdgcn_global_load_lds" not in code(name):
            continue
        text = code(name)
        for m in re.finditer(r"void\s+(\w+)\s*\([^;{]*\)\s*(?=\{)", text):
            b = body(text, m.end())
            at = b.find("__builtin_amdgcn_global_load_lds")
            if at < 0:
                continue
            found += 1
            wait = re.search(r"s_waitcnt[^\"]*lgkmcnt\(0\)|__builtin_amdgcn_s_waitcnt\(kWaitLds\)", b)
            assert wait and wait.start() < at, f"{name}: {m.group(1)}"
    assert found >= 1
    # vmcnt and expcnt at their largest, lgkmcnt 0
    assert re.search(r"kWaitLds = 0xc07f;", code("lw_fused.hip"))


def test_row_map_reads_stay_within_the_coupled_rows():
    """The LU's row map holds n entries; a block of 64 rows may end past them, so every read of
    it is clamped to n - 1."""
    text = code("bte.hip")
    lu = text[text.index("lu_panels"):text.index("lu_gemm(")]
    reads = re.findall(r"A\.rows\[([^\]]*)\]", lu)
    assert len(reads) >= 3
    for r in reads:
        assert re.match(r"min\(.*, n - 1\)$", r), r
