"""The launch plan on the GPU: small tiles of the builds with run-time offsets keep the workgroups
per CU that their LDS leaves room for (the kernels' registers must not lower it), so that a
mesh of one tile per such workgroup runs as one resident launch."""
import numpy as np
import pytest

from paper_2005_02516_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _info(w, precision, **kw):
    from paper_2005_02516_amd.binding import EsdgSwe
    s = EsdgSwe([w], precision=precision, flux="lf", g=w.g, **kw)
    info = s.launch_info()
    s.close()
    return info


# elements per tile, workgroups per CU (registers of at most 96 a lane five, 80 six of 256
# threads or three of 512)
@pytest.mark.parametrize("N,precision,mass,E,per_cu", [
    (3, "fp32", "stored", 4, 5), (3, "fp32", "wadg", 4, 5), (2, "fp64", "stored", 4, 5), (2, "fp64", "wadg", 4, 5),
    (4, "fp32", "wadg", 4, 5), (4, "fp32", "stored", 2, 6), (5, "fp32", "stored", 2, 3)])
def test_small_tiles_stay_resident(torch_mod, N, precision, mass, E, per_cu):
    cus = torch_mod.cuda.get_device_properties(0).multi_processor_count
    n = int((per_cu * cus * E // 2) ** 0.5)          # 2 n^2 elements: at most one tile per workgroup
    info = _info(wl.config2(n=n, N=N), precision, mass=mass, elems_per_block=E)
    print(N, precision, mass, E, info, flush=True)
    assert info["resident_workgroups"] >= per_cu * cus, info
    assert info["step_mode"] == 2, info
