"""Tile sizes on the GPU: the sizes with kernels of their own, one less (run-time offsets), one
element, and tiles larger than the mesh, all with ragged last tiles (32 elements), each kind
and precision.  One RHS within 64 eps of its forward rounding bound against the oracle
(parity_util), the no-allocation RHS bitwise equal to it, and steps in one multi-stage launch
bitwise equal to one launch per stage.  Launches of several degrees with more tiles than
workgroups (split by cost): FP64 steps to 1e-12 of each mesh's own solver."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

from oracle import esdg_oracle as O
from paper_2005_02516_amd import sbp_rules
from paper_2005_02516_amd import workloads as wl
from parity_util import EPS32, EPS64, check_rhs, rhs_abs_bound, sbp_rhs_abs_bound

pytestmark = pytest.mark.gpu

FP32 = {1: (32, 16), 2: (14, 12), 3: (8,), 4: (5,), 5: (7,)}
FP64 = {1: (16, 12), 2: (7, 8), 3: (4,), 4: (5,), 5: (7,)}
SBP32 = {1: (16,), 2: (13,), 3: (8,), 4: (8,)}
SBP64 = {1: (8,), 2: (8,), 3: (4,), 4: (4,)}


def _cases(sizes):
    for N, own in sizes.items():
        for E in sorted({1, *own, *(e - 1 for e in own)} - {0}):
            yield N, E


def _moving(w):
    rng = np.random.default_rng(w.N)
    u = w.u_nodes.copy()
    u[1] += 0.1 * u[0] * rng.uniform(-1, 1, u[0].shape)
    u[2] += 0.1 * u[0] * rng.uniform(-1, 1, u[0].shape)
    return u


def _solver(ws, precision, **kw):
    from paper_2005_02516_amd.binding import EsdgSwe
    s = EsdgSwe(ws, precision=precision, flux="lf", g=ws[0].g, **kw)
    for i, w in enumerate(ws):
        s.set_state(i, _moving(w))
    return s


def _rhs(torch, s):
    st = s.state_device(0)
    out, free = torch.empty_like(st), torch.empty_like(st)
    s.rhs(0, st, out)
    s.rhs_noalloc(0, st, free)
    s.sync()
    assert torch.equal(out, free)
    return out.cpu().double().numpy(), s.get_state(0)


def _steps(ws, precision, steps, **kw):
    s = _solver(ws, precision, **kw)
    s.step(np.array([w.dt for w in ws]), steps)
    out = [s.get_state(i) for i in range(len(ws))]
    s.close()
    return out


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("mass", ["stored", "wadg"])
def test_modal_tiles(torch_mod, precision, mass):
    for N, E in _cases(FP32 if precision == "fp32" else FP64):
        print(f"modal N={N} E={E} {precision} {mass}", flush=True)
        w = wl.config2(n=4, N=N)
        s = _solver([w], precision, elems_per_block=E, mass=mass)
        r, uh = _rhs(torch_mod, s)
        s.close()
        o = O.Oracle(O.Discretization(N, w.xg, w.yg, w.b_nodes, w.g, w.Lx, w.Ly,
                                      mass="exact" if mass == "stored" else mass), "lf")
        ok, worst = check_rhs(r, o.rhs(uh), rhs_abs_bound(o, uh, np.arange(w.K)), EPS32 if precision == "fp32" else EPS64)
        assert ok, (N, E, worst)
        ref, got = (_steps([w], precision, 3, elems_per_block=E, mass=mass, fused=f) for f in (False, True))
        assert np.array_equal(ref[0], got[0]), (N, E)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_sbp_tiles(torch_mod, precision):
    for N, E in _cases(SBP32 if precision == "fp32" else SBP64):
        print(f"DG-SBP N={N} E={E} {precision}", flush=True)
        w = wl.config2(n=4, N=N)
        rule = {"rule": sbp_rules.load(N)}
        s = _solver([w], precision, elems_per_block=E, scheme="sbp", quadrature=rule)
        r, u = _rhs(torch_mod, s)
        s.close()
        o = O.SBPOracle(O.Discretization(N, w.xg, w.yg, w.b_nodes, w.g, w.Lx, w.Ly,
                                         quad={**rule, "vol_degree": 2 * N - 1}), "lf")
        ok, worst = check_rhs(r, o.rhs(u), sbp_rhs_abs_bound(o, u), EPS32 if precision == "fp32" else EPS64)
        assert ok, (N, E, worst)


@pytest.mark.parametrize("epb", [None, {1: 1, 2: 1, 3: 1}])
def test_mixed_split(torch_mod, epb):
    ws = [wl.config2(n=n, N=N) for N, n in ((1, 40), (2, 3), (1, 3), (3, 8), (2, 24))]
    got = _steps(ws, "fp64", 3, elems_per_block=epb, fused=False)
    for w, u in zip(ws, got):
        ref = _steps([w], "fp64", 3, fused=False)[0]
        scale = np.abs(ref[0]).max()
        assert np.abs(u - ref).max() < 1e-12 * scale, (w.N, w.K)
