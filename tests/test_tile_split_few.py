"""The tile cut where units are few: up to one unit per CU, every tile is one unit,
also where humans' odd halves would otherwise be the largest tiles (no GPU)."""
import numpy as np
import pytest


@pytest.mark.parametrize("C", [8, 255, 256])
@pytest.mark.parametrize("rem", [0, 1, 2, 3])
def test_few_units_are_single(C, rem):
    from paper_2603_01122_amd import capred
    r = np.random.default_rng(C + rem)
    for R in (C, 2 * C, 3 * C):
        for _ in range(20):
            units = 4 * r.integers(0, 3, size=int(r.integers(1, 12))) + rem
            while units.sum() > C:
                units = units[:-1]
            cnt = capred.tile_split(units, 4, R, C)
            assert np.array_equal(cnt @ np.array([4, 2, 1]), units)
            assert cnt[:, 0].sum() == 0 and cnt[:, 1].sum() <= 1
