"""Inline assembly of the kernels: a statement that writes m0 says so to the compiler."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_07173_amd", "csrc")


def test_writes_of_m0_are_declared():
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        for m in re.finditer(r"\basm\b[^;]*;", open(path, errors="replace").read()):
            if re.search(r"\bs_\w+ +m0\b", m.group(0)):
                found += 1
                assert re.search(r':[^:]*"m0"[^:]*\)\s*;$', m.group(0)), f"{os.path.basename(path)}: {m.group(0)}"
    assert found == 2
