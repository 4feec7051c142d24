"""FP32 rounding of a right-hand side against the FP64 oracle on the same (float) state, as an RMS
over all values relative to the RMS of the result.

The products with the constant operators add their terms in two chains, and the interface
terms enter one of the residual's two parts, so that no sum is longer than in the scheme's
first kernels (vector ALUs, two partial sums each).  With one chain the error of these kinds is
8 to 13 % larger.  REFERENCE holds the error of those first kernels on the same inputs; the bar
is 4 % above it, four times the spread of the ratio between seeds (1 %)."""
import numpy as np
import pytest

from oracle import esdg_oracle as O
from paper_2005_02516_amd import workloads as wl

pytestmark = pytest.mark.gpu

REFERENCE = {(4, "wadg", False): 3.2256e-07, (5, "wadg", False): 4.1223e-07, (2, "stored", True): 1.7728e-07,
             (3, "stored", True): 2.0817e-07, (4, "stored", True): 2.7383e-07, (5, "stored", True): 3.1023e-07}


def kinds():
    for N in (4, 5):
        yield N, "wadg", False
    for N in (2, 3, 4, 5):
        yield N, "stored", True


def rms_error(torch, N, mass, plus, seeds=4):
    from paper_2005_02516_amd.binding import EsdgSwe
    w = wl.config2(n=16, N=N)
    quad = {"vol_degree": 2 * N + 2, "face_points": N + 2} if plus else None
    o = O.Oracle(O.Discretization(N, w.xg, w.yg, w.b_nodes, w.g, w.Lx, w.Ly, quad=quad,
                                  mass="exact" if mass == "stored" else mass), "lf")
    s = EsdgSwe([w], precision="fp32", flux="lf", g=w.g, mass=mass, quadrature=quad)
    err = []
    for seed in range(seeds):
        rng = np.random.default_rng(seed)
        u = w.u_nodes.copy()
        u[1] += 0.1 * u[0] * rng.uniform(-1, 1, u[0].shape)
        u[2] += 0.1 * u[0] * rng.uniform(-1, 1, u[0].shape)
        s.set_state(0, u)
        st = s.state_device(0)
        out = torch.empty_like(st)
        s.rhs(0, st, out)
        s.sync()
        ref = o.rhs(s.get_state(0))
        d = out.cpu().double().numpy() - ref
        err.append(np.sqrt(np.mean(d * d) / np.mean(ref * ref)))
    s.close()
    return float(np.exp(np.mean(np.log(err))))


@pytest.mark.parametrize("N,mass,plus", list(kinds()))
def test_rhs_rounding(torch_mod, N, mass, plus):
    e = rms_error(torch_mod, N, mass, plus)
    print(f"N={N} {mass} plus={plus}: {e:.4e}", flush=True)
    assert e <= 1.04 * REFERENCE[N, mass, plus], e / REFERENCE[N, mass, plus]
