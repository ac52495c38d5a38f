"""The autotuner's cache file (host) and the settings it tunes under (GPU)."""
import json

import pytest

import paper_1709_09713_amd as ns
from paper_1709_09713_amd import _native as nat
from paper_1709_09713_amd.autotune import Autotuner


def test_entries_hold_for_the_build_they_were_tuned_with(tmp_path, monkeypatch):
    path = str(tmp_path / "tuned.json")
    calls = []

    def tune(self, n, precision):
        calls.append((n, precision))
        return {"tile": 3, "zchunk": 5}

    monkeypatch.setattr(Autotuner, "tune", tune)
    with open(path, "w") as f:   # of another build, and of one that kept no name
        json.dump({"16x16x16:fp64": {"tile": 8, "zchunk": 6, "library": "0" * 16},
                   "24x24x24:fp32": {"tile": 8, "zchunk": 6}}, f)
    a = Autotuner(path)
    assert a.lookup(16, "fp64") == (3, 5) and a.lookup(24, "fp32") == (3, 5)
    assert a.lookup(16, "fp64") == (3, 5) and len(calls) == 2
    assert Autotuner(path).lookup((16, 16, 16), "fp64") == (3, 5) and len(calls) == 2


@pytest.mark.gpu
def test_tuning_ignores_the_callers_settings(monkeypatch):
    p = nat.make_params(20)
    default = nat.ns_get_fused_config(p)
    add = nat.ns_batch_add
    seen = []

    def record(*args, **kw):
        seen.append(nat.ns_get_fused_config(p))
        return add(*args, **kw)

    monkeypatch.setattr(nat, "ns_batch_add", record)
    ns.ns_set_fused_config(4, 7)
    try:
        Autotuner(tiles=(-1, 9), zchunks=(0,), steps=1, reps=1).tune(20, "fp64")
        assert nat.ns_get_fused_config(p) == (4, 7)
    finally:
        ns.ns_set_fused_config(-1, 0)
    assert len(seen) == 2 and all(s == default for s in seen)
