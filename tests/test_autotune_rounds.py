"""Tile sizes by rounds of resident workgroups (CPU): a size that a class of meshes takes can need
one round more than another between two sizes, and then another one is faster."""
import json

import pytest

from paper_2005_02516_amd import autotune as A


def test_best_by_rounds():
    table = {"7": [512, 10.0, 8.0], "16": [256, 16.0, 15.0]}
    assert A.best_by_rounds(table, [7 * 512]) == 7                 # resident: 8 against 15
    assert A.best_by_rounds(table, [7 * 512 + 1]) == 16            # two rounds of 10 against 15
    assert A.best_by_rounds(table, [16 * 256]) == 16
    assert A.best_by_rounds(table, [16 * 256 + 1]) == 7            # two rounds each
    assert A.best_by_rounds(table, [1] * 257) == 7                 # a tile for each mesh
    assert A.best_by_rounds(table, [8] * 256 + [17]) == 7


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
def test_n5_between_the_tile_sizes(precision):
    """N = 5: 16 elements to a tile where they leave one tile per workgroup and 7 do not, which is
    what the class took before 7 became its size; 7 below and above."""
    look = lambda K, **kw: A.lookup_shapes(precision, [(5, K)], **kw)[0][5]  # noqa: E731
    assert [look(K) for K in (32, 3584, 3585, 4050, 4096, 4097, 10000)] == [7, 7, 16, 16, 16, 7, 7]
    assert look(8192) == (16 if precision == "bf16x3" else 7)
    assert look(4050, mass="wadg") == 7            # another LDS need: the table does not apply
    assert A.lookup(precision, [(5, 4050), (2, 100)])[5] <= 7


def test_n1_fp64_large_meshes():
    """FP64 N = 1 from 32768 elements on: 12 elements to a tile with the stored inverse, six
    workgroups a CU; 16 with the weight-adjusted one and next to other degrees, as before."""
    for K in (32768, 45000, 65522, 131072, 262143):
        assert A.lookup("fp64", [(1, K)]) == {1: 12}
        assert A.lookup_shapes("fp64", [(1, K)], mass="wadg")[0] == {1: 16}
    assert A.lookup("fp64", [(1, 8192)]) == {1: 16}


def test_rounds_tables_are_timed_sizes():
    with open(A.CACHE) as f:
        for key, e in json.load(f)["entries"].items():
            for table in e.get("rounds", {}).values():
                assert str(e["epb"]) in table, key
                for E, (blocks, each, resident) in table.items():
                    assert E in e["us_per_stage"] and blocks % 256 == 0 and 0 < resident < each, (key, E)


def test_tune_times_no_shapes(monkeypatch):
    """The tuner times each E once, with the default shape, and keeps a rounds table."""
    seen = []
    monkeypatch.setattr(A, "time_config", lambda w, p, E, steps=4, warmup=1, shape=None: seen.append((E, shape)) or 1.0 / E)
    data = A.tune([(5, 4)], precisions=("fp32",), write=False, log=open("/dev/null", "w"))
    e = data["entries"]["fp32:N5:S"]
    assert len(seen) == len(set(seen)) and {s for _, s in seen} == {None}
    assert e["epb"] == max(E for E, _ in seen) and "rows" not in e and "rounds" in e
    data = A.tune([(1, 128)], precisions=("fp64",), write=False, log=open("/dev/null", "w"))
    assert data["entries"]["fp64:N1:M"]["epb_else"] == 16
