"""Host-side checks of the kernel sources and of the index and planning helpers that kernels and
runtime share (CPU; the headers are compiled with g++)."""
import os
import re
import subprocess

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


def _run_cpp(tmp_path, body, includes=("device_types.hpp",)):
    """The standard output of a program compiled with g++ against the named headers."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text("#include <cstdio>\n#include <vector>\n" + "".join(f'#include "{h}"\n' for h in includes) +
                   "using namespace esdg;\nint main() {\n" + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


def test_progress_words_do_not_wrap(tmp_path):
    """The words of the progress counts of 2^26 tiles and more lie beyond 32 bits."""
    out = _run_cpp(tmp_path, """for (int t : {0, 1, (1 << 26) - 1, 1 << 26, 0x7fffffff})
  std::printf("%llu ", (unsigned long long)progress_word(t));""")
    assert [int(v) for v in out.split()] == [32 * t for t in (0, 1, 2**26 - 1, 2**26, 2**31 - 1)]
    text = open(os.path.join(CSRC, "kernels.hip")).read()
    assert not re.search(r"progress \+ (?!progress_word)", text)
