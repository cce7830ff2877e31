"""Inline assembly of the kernels: a statement that writes a register names it as an output or clobber."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2211_09370_amd", "csrc")


def test_statements_that_write_m0_name_it():
    found = 0
    for path in glob.glob(os.path.join(CSRC, "*")):
        for text in re.findall(r"asm volatile\((.*?)\);", open(path, errors="replace").read(), flags=re.S):
            if re.search(r"s_mov_b32 m0", text):
                found += 1
                clobbers = text.rsplit(":", 1)[1]
                assert '"m0"' in clobbers, (os.path.basename(path), text)
    assert found >= 2
