"""Which LU a sweep sizes its chunks and parts for (host only)."""
import types

import numpy as np
import pytest

from paper_1902_01458_amd import api


class Sized(Exception):
    pass


# (tune, tile that factor_bytes has to be asked for)
CASES = [(None, 0), ({"tile": 32, "grid": 7}, 0), ({"tile": 64, "grid": 7, "superblock": 0}, 0),
         ({"tile": 32, "grid": 7, "superblock": 4}, 32),
         ({"tile": 0, "grid": 0, "superblock": 4}, 64), ({"tile": 0, "grid": 0, "superblock": -1}, 64)]


@pytest.mark.parametrize("tune,want", CASES)
def test_chunks_and_parts_are_sized_for_the_lu_they_get(monkeypatch, tune, want):
    prob = types.SimpleNamespace(nx=512, ny=256, n=2 * 512 * 256)
    asked = []

    def chunk_size(prob, k, precision, tile, *_):
        asked.append(tile)
        raise Sized

    monkeypatch.setattr(api, "_chunk_size", chunk_size)
    with pytest.raises(Sized):
        api.sweep(prob, [1.0, 2.0], 20, tune=tune)

    def factor_bytes(nx, ny, n_omega, k, precision, tile):
        asked.append(tile)
        return 1

    def factor(prob, om, precision, k_max, tile, grid, superblock):
        raise Sized

    monkeypatch.setattr(api, "factor_bytes", factor_bytes)
    monkeypatch.setattr(api, "factor", factor)
    t = tune or {"tile": 0, "grid": 0}
    with pytest.raises(Sized):
        api._sweep_chunk(prob, np.array([1.0, 2.0]), 20, 0, 0, "fp64", t["tile"], t["grid"],
                         t.get("superblock", 0))
    assert asked == [want, want]


def test_the_band_is_the_larger_of_the_two():
    """What a chunk sized for the wrong LU would run out of."""
    one = api.factor_bytes(512, 256, 1, 20, "fp64", 0)
    assert api.factor_bytes(512, 256, 1, 20, "fp64", 64) > 3 * one > 0
