"""Host-side checks of the kernel sources and of the index and planning helpers that kernels and
runtime share (CPU; the headers are compiled with g++)."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_02516_amd", "csrc")


def _asm_statements(text):
    for m in re.finditer(r"\basm\s+volatile\s*\(", text):
        depth, i = 1, m.end()
        quoted = False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(c, 0)
            i += 1
        yield text[m.end():i - 1]


def test_asm_that_writes_m0_says_so():
    """Inline asm that sets M0 names it as clobbered: the compiler may otherwise keep a value of its
    own there across the statement."""
    seen = 0
    for f in sorted(os.listdir(CSRC)):
        for s in _asm_statements(open(os.path.join(CSRC, f)).read()):
            if re.search(r"\bm0\s*,", s):
                seen += 1
                assert re.search(r':[^:]*"m0"[^:]*$', s), (f, s)
    assert seen >= 3
