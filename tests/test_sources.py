"""Checks on the kernels' sources that need neither a compiler nor a GPU."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_09360_amd", "csrc")


def test_inline_assembly_declares_the_m0_it_writes():
    """The compiler keeps values of its own in m0 (indexed register and LDS forms): an assembly statement that writes it
    has to say so."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        for stmt in re.findall(r"\basm\b[^;]*?\((.*?)\)\s*;", open(path).read(), flags=re.S):
            template = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', stmt.split(":")[0]))
            if re.search(r"\bs_\w+\s+m0\b", template):
                seen += 1
                assert '"m0"' in stmt.split(":")[-1], (os.path.basename(path), template)
    assert seen > 0
