"""What the tuner times and how a tile size is chosen from it (CPU)."""
from paper_2005_02516_amd import autotune as A


def test_tune_times_no_shapes(monkeypatch):
    """The tuner times each E once, with the default shape, and names no shape."""
    seen = []
    monkeypatch.setattr(A, "time_config", lambda w, p, E, steps=4, warmup=1, shape=None: seen.append((E, shape)) or 1.0 / E)
    data = A.tune([(5, 4)], precisions=("fp32",), write=False, log=open("/dev/null", "w"))
    e = data["entries"]["fp32:N5:S"]
    assert len(seen) == len(set(seen)) and {s for _, s in seen} == {None}
    assert e["epb"] == max(E for E, _ in seen) and "rows" not in e
