"""The cube lattice's faces: a boundary coordinate is 0 or 1 exactly and stays there, also for the sides m whose
m (1 / m) rounds below 1 (49, 98, 103, 107 are the first), so that every mesh lies in the unit cube. 48, 50 and 100 are
sides where it rounds to 1: their points are as the product gives them."""
import numpy as np
import pytest

from paper_1209_5421_amd import meshgen as mg


@pytest.mark.parametrize("m", [48, 49, 50])
def test_faces_stay_on_the_cube(m):
    pts, tets, inlet = mg.cube_mesh(m)
    assert pts.min() == 0.0 and pts.max() == 1.0
    assert int(inlet.sum()) == (m + 1) ** 2
    for axis in range(3):
        assert int((pts[:, axis] == 0.0).sum()) == (m + 1) ** 2
        assert int((pts[:, axis] == 1.0).sum()) == (m + 1) ** 2
    assert len(tets) == 6 * m ** 3


def test_sides_that_round_low_are_the_ones_named():
    low = [m for m in range(1, 108) if m * (1.0 / m) < 1.0]
    assert low == [49, 98, 103, 107]
    assert 48 * (1.0 / 48) == 1.0 and 50 * (1.0 / 50) == 1.0 and 100 * (1.0 / 100) == 1.0
