"""The launch plan on the GPU: small tiles of the builds with run-time offsets keep the workgroups
per CU that their LDS leaves room for (the kernels' registers must not lower it), so that a
mesh of one tile per such workgroup runs as one resident launch; the tile shape option does
not enter it."""
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


@pytest.mark.parametrize("N,precision,E", [(1, "fp32", 48), (2, "fp32", 14), (3, "fp32", 8), (4, "fp32", 5), (4, "fp64", 3),
                                           (5, "fp32", 6)])
def test_tile_shape_leaves_the_plan(torch_mod, N, precision, E):
    """The tile shape enters the limit of elems_per_block only: every accepted one gives the
    same workgroups, LDS and step mode."""
    from paper_2005_02516_amd.autotune import shapes
    from paper_2005_02516_amd.binding import shape_code
    w = wl.config2(n=8, N=N)
    ref = _info(w, precision, elems_per_block=E)
    for R, P in shapes(N, precision):
        assert _info(w, precision, elems_per_block=E, tile_shape=shape_code(R, P)) == ref, (R, P)


@pytest.mark.parametrize("precision,N,E,words_bytes,per_cu", [
    ("fp32", 1, 36, 40880, 3), ("fp32", 1, 48, 54272, 2), ("fp32", 2, 25, 54196, 2), ("fp64", 1, 36, 81760, 1)])
def test_plan_counts_static_lds_in_granules(torch_mod, precision, N, E, words_bytes, per_cu):
    """Tile sizes whose counted LDS fits 160 KiB once more without the multi-stage build's own 256
    bytes or the 1 KiB granules: the plan counts both."""
    from paper_2005_02516_amd import autotune as A
    word = 8 if precision == "fp64" else 4
    assert (A.ref_words(N) + A.tile_words(N, E, A.default_shape(N, precision)[1])) * word == words_bytes
    assert 160 * 1024 // words_bytes == per_cu + 1
    cus = torch_mod.cuda.get_device_properties(0).multi_processor_count
    info = _info(wl.config2(n=8, N=N), precision, elems_per_block=E)
    assert info["resident_workgroups"] == per_cu * cus, info
