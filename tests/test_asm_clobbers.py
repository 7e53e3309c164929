"""Inline assembly that writes M0 says so, so that no value of the compiler's
lives there across it."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_03868_amd", "csrc")


def test_m0_is_declared():
    seen = 0
    for path in glob.glob(os.path.join(CSRC, "*.h*")):
        for stmt in re.findall(r"asm volatile\(.*?\);", open(path).read(), re.S):
            if re.search(r"\bm0,", stmt):
                seen += 1
                clobbers = stmt.rsplit(":", 1)[1]
                assert '"m0"' in clobbers and '"memory"' in clobbers, (path, stmt)
    assert seen >= 4
