"""Inline assembly states every register it writes: the compiler keeps its own values in those it is not told about."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_18164_amd", "csrc")


def statements():
    for name in sorted(os.listdir(CSRC)):
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\((.*?)\)\s*;", open(os.path.join(CSRC, name)).read(), re.S):
            yield name, m.group(1)


def test_statements_that_write_m0_say_so():
    writes = [(name, s) for name, s in statements() if re.search(r"s_\w+\s+m0\b", s)]
    assert writes                                        # the direct loads to LDS take their address from it
    for name, s in writes:
        assert re.search(r':[^:]*"m0"[^:]*$', s), (name, s)
