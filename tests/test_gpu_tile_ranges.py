"""Launches of several degrees with more tiles than workgroups, whose tiles are split by cost into
uneven ranges, and ragged tiles, on the GPU.

The kernel for several degrees with fixed tile sizes and the one with run-time offsets, FP32 and
FP64: steps in one multi-stage launch bitwise equal to one launch per stage, and both within 64 eps
of the largest value of each mesh's own solver with the same tiles (the sums run in the same
order; the bar leaves room for a few roundings that do not).

Every tile size with a kernel of its own on meshes that it does not divide, and that are smaller
than one tile: one RHS within 64 eps of its forward rounding bound against the oracle, the
no-allocation RHS bitwise equal to it, steps in one multi-stage launch bitwise equal to per-stage
launches."""
import numpy as np
import pytest

from oracle import esdg_oracle as O
from paper_2005_02516_amd import sbp_rules
from paper_2005_02516_amd import workloads as wl
from parity_util import EPS32, EPS64, check_rhs, rhs_abs_bound, sbp_rhs_abs_bound
from test_gpu_tiles import FP32, FP64, SBP32, SBP64, _rhs, _solver, _steps

pytestmark = pytest.mark.gpu


def _meshes(cus, epb):
    """Meshes of the degrees of epb in mixed order with about seven tiles per CU, all ragged."""
    shares = [(s, N) for s, N in ((3, 3), (1, 2), (2, 4), (1, 1), (1, 2)) if N in epb]
    out = []
    for share, N in shares:
        n = int((7 * cus * share / sum(s for s, _ in shares) * epb[N] / 2) ** 0.5) | 1
        while 2 * n * n % epb[N] == 0:
            n += 2
        out.append(wl.config2(n=n, N=N))
    return out


# the fixed sizes of both kinds of N = 1 and 2, and sizes that take run-time offsets
@pytest.mark.parametrize("precision,epb", [
    ("fp32", {1: 32, 2: 14, 3: 8, 4: 5}), ("fp32", {1: 16, 2: 12, 3: 8, 4: 5}), ("fp32", {2: 10, 3: 4}),
    ("fp64", {1: 16, 2: 7, 3: 4}), ("fp64", {1: 12, 2: 8, 3: 4, 4: 5}), ("fp64", {2: 5, 3: 3})])
def test_uneven_ranges(torch_mod, precision, epb):
    cus = torch_mod.cuda.get_device_properties(0).multi_processor_count
    ws = _meshes(cus, epb)
    assert all(w.K % epb[w.N] for w in ws)
    s = _solver(ws, precision, elems_per_block=epb, fused=True)
    info = s.launch_info()
    s.close()
    print(precision, epb, info, flush=True)
    assert info["step_mode"] == 1 and info["tiles"] > info["resident_workgroups"], info
    per_stage, multi = (_steps(ws, precision, 2, elems_per_block=epb, fused=f) for f in (False, True))
    eps = EPS32 if precision == "fp32" else EPS64
    for w, a, b in zip(ws, per_stage, multi):
        assert np.array_equal(a, b), (w.N, w.K)
        own = _steps([w], precision, 2, elems_per_block=epb, fused=False)[0]
        assert np.abs(a - own).max() <= 64 * eps * np.abs(own).max(), (w.N, w.K)


def _ragged(sizes, n, odd):
    """(N, E, mesh) for every size: n squares a side, or the first odd number from there on whose
    mesh the size does not divide."""
    for N, own in sizes.items():
        for E in own:
            m = n
            while odd and 2 * m * m % E == 0:
                m += 2
            yield N, E, wl.config2(n=m, N=N)


@pytest.mark.parametrize("n", [1, 3, 5])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("mass", ["stored", "wadg"])
def test_modal_ragged(torch_mod, precision, mass, n):
    eps = EPS32 if precision == "fp32" else EPS64
    for N, E, w in _ragged(FP32 if precision == "fp32" else FP64, n, n > 1):
        print(f"modal N={N} E={E} K={w.K} {precision} {mass}", flush=True)
        assert w.K % E or w.K < E
        s = _solver([w], precision, elems_per_block=E, mass=mass)
        r, uh = _rhs(torch_mod, s)
        s.close()
        o = O.Oracle(O.Discretization(N, w.xg, w.yg, w.b_nodes, w.g, w.Lx, w.Ly,
                                      mass="exact" if mass == "stored" else mass), "lf")
        ok, worst = check_rhs(r, o.rhs(uh), rhs_abs_bound(o, uh, np.arange(w.K)), eps)
        assert ok, (N, E, w.K, worst)
        ref, got = (_steps([w], precision, 3, elems_per_block=E, mass=mass, fused=f) for f in (False, True))
        assert np.array_equal(ref[0], got[0]), (N, E, w.K)


@pytest.mark.parametrize("n", [1, 3, 5])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_sbp_ragged(torch_mod, precision, n):
    eps = EPS32 if precision == "fp32" else EPS64
    for N, E, w in _ragged(SBP32 if precision == "fp32" else SBP64, n, n > 1):
        print(f"DG-SBP N={N} E={E} K={w.K} {precision}", flush=True)
        assert w.K % E or w.K < E
        rule = {"rule": sbp_rules.load(N)}
        s = _solver([w], precision, elems_per_block=E, scheme="sbp", quadrature=rule)
        r, u = _rhs(torch_mod, s)
        s.close()
        o = O.SBPOracle(O.Discretization(N, w.xg, w.yg, w.b_nodes, w.g, w.Lx, w.Ly,
                                         quad={**rule, "vol_degree": 2 * N - 1}), "lf")
        ok, worst = check_rhs(r, o.rhs(u), sbp_rhs_abs_bound(o, u), eps)
        assert ok, (N, E, w.K, worst)
