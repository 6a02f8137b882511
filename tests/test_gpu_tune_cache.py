"""The autotuner's cache file: which entries are taken."""
import json

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def rr():
    import paper_1902_01458_amd as m
    return m


def test_a_pick_from_the_band_only_candidates_is_not_taken(tmp_path, monkeypatch):
    """A file written when the band LU was the only candidate: the trials run
    again, and their pick stands beside the old entry; a later call takes it."""
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("RR_AUTOTUNE_CACHE", str(cache))
    w = W.small("atc", 40, 32, nu=1e-2, omegas=(0.6, 2.2), k=8, q=0)
    prob = rr().BurgersProblem.from_workload(w)
    old = {"tile": 32, "grid": 7, "superblock": 8, "ms": 0.001}
    cache.write_text('{\n"gfx950|40x32|w2|k8|fp64": ' + json.dumps(old) + "\n}\n")
    pick = rr().autotune(prob, list(w.omegas), w.k, "fp64")
    assert pick["grid"] != 7 and pick["ms"] > 0.001
    entries = json.loads(cache.read_text())
    assert entries["gfx950|40x32|w2|k8|fp64"] == old and len(entries) == 2
    assert rr().autotune(prob, list(w.omegas), w.k, "fp64") == pick
