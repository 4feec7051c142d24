"""Host-side checks of the kernel sources and of the index and planning helpers that kernels and
runtime share (CPU; the headers are compiled with g++)."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2005_02516_amd import binding, sbp_rules
from paper_2005_02516_amd import workloads as wl

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


def _workspace(w, E, **kw):
    lib = binding.load_library()
    scheme = kw.pop("scheme", "modal")
    xg, yg, b = (np.ascontiguousarray(a) for a in (w.xg, w.yg, w.b_nodes))
    arr = (binding.esdg_swe_instance * 1)()
    arr[0] = binding.esdg_swe_instance(w.N, w.K, binding._dptr(xg), binding._dptr(yg), binding._dptr(b), w.Lx, w.Ly)
    keep = []
    q = (binding.esdg_swe_quadrature * 1)()
    q[0] = binding.make_quadrature({"rule": sbp_rules.load(w.N)} if scheme == "sbp" else None, keep)
    opt = binding.make_options("fp32", "lf", 1.0, True, {w.N: E}, scheme=scheme, **kw)
    h, nb = C.c_void_p(), C.c_size_t()
    assert lib.esdg_swe_init(1, arr, q, C.byref(opt), C.byref(h), C.byref(nb)) == binding.ESDG_OK
    lib.esdg_swe_destroy(h)
    return nb.value


@pytest.mark.parametrize("n", [20, 50])
def test_progress_counts_only_where_used(n):
    """The workspace has a 128-byte line per tile for plans that may be one launch per step call
    (forced, or automatic with at most 2048 tiles), and none for the others."""
    w = wl.config2(n=n, N=1)
    tiles = w.K                                    # one element each
    off, auto, forced = (_workspace(w, 1, fused=f) for f in (False, "auto", True))
    assert forced - off == 128 * tiles
    assert auto == (forced if tiles <= 2048 else off)
    assert _workspace(w, 1, scheme="sbp", fused=True) == _workspace(w, 1, scheme="sbp", fused=False)
    # DG-SBP: what a tile more costs (tile, descriptors, padding) is less than a line
    a, b = (_workspace(w, E, scheme="sbp") for E in (1, 2))
    assert a - b < 128 * (tiles - tiles // 2)


def _smallest_largest(cost, G):
    """The smallest possible cost of the largest of G contiguous ranges, by dynamic programming."""
    n = len(cost)
    best = [sum(cost[:i]) for i in range(n + 1)]           # one range
    for _ in range(G - 1):
        best = [min(max(best[j], sum(cost[j:i])) for j in range(i + 1)) for i in range(n + 1)]
    return best[n]


def test_split_tiles(tmp_path):
    """The ranges cover every tile once, in order, and their largest cost is the smallest possible."""
    rng = np.random.default_rng(7)
    cases = [([int(c) for c in rng.integers(1, hi, rng.integers(1, 13))], int(rng.integers(1, 9)))
             for hi in (2, 4, 60, 600) for _ in range(40)]
    cases += [([5] * 12, 12), ([1, 1, 1, 100], 3), ([100, 1, 1, 1], 3), ([7], 8)]
    body = ""
    for cost, G in cases:
        cum = np.concatenate([[0], np.cumsum(cost)])
        body += f"for (int v : split_tiles({{{', '.join(str(c) for c in cum)}}}, {G})) std::printf(\"%d \", v);\n"
        body += 'std::printf("\\n");\n'
    rows = _run_cpp(tmp_path, body, ("tile_plan.hpp",)).splitlines()
    assert len(rows) == len(cases)
    for (cost, G), row in zip(cases, rows):
        r = [int(v) for v in row.split()]
        assert len(r) == G + 1 and r[0] == 0 and r[G] == len(cost) and r == sorted(r), (cost, G, r)
        assert max(sum(cost[a:b]) for a, b in zip(r, r[1:])) == _smallest_largest(cost, G), (cost, G, r)


def test_tile_ranges_only_where_tiles_differ(tmp_path):
    """No ranges for one kind, nor with a workgroup for every tile; bind takes what a launch uses from
    this answer, so that a second bind cannot keep ranges its workspace does not hold."""
    out = _run_cpp(tmp_path, """std::vector<long long> cum = {0, 3, 5, 6, 10};
std::printf("%d %d %d %d %d", int(tile_ranges(cum, 1, 2).size()), int(tile_ranges(cum, 2, 4).size()),
            int(tile_ranges(cum, 2, 8).size()), int(tile_ranges(cum, 2, 3).size()), int(tile_ranges({0}, 1, 8).size()));""",
                   ("tile_plan.hpp",))
    assert out.split() == ["0", "0", "0", "4", "0"]
    text = open(os.path.join(CSRC, "runtime.cpp")).read()
    assert re.findall(r"balanced = ([^;]*);", text) == ["false", "!ranges.empty()"]
