"""Uneven spots, and small spots of many shapes, in the passes made for them.

Batches of one uneven shape branch over the row tiles below their spots (32 and 64
spots per wavefront), spots of any shapes up to 8 x 8 go through passes of two
tiles, and a few wide floats have passes with four tiles one way: each gives the bits
of the passes for mixed shapes (16 spots per wavefront), which the other tests hold
against the oracle."""
import os

import numpy as np
import pytest

from test_gpu_matrix import _equal, _fit, _shapes

pytestmark = pytest.mark.gpu

TILES = [(3, 32), (32, 3), (4, 32), (5, 29), (29, 5), (30, 12), (12, 30), (16, 17), (17, 16), (20, 25), (28, 32),
         (32, 28), (7, 16), (16, 7), (4, 13), (13, 4), (9, 12), (16, 4)]


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("slots", [32, 64])
def test_one_uneven_shape(slots, f32):
    """Every spot in turn is new, accepted and retried beside others; a ragged last pass."""
    for i, (w, h) in enumerate(TILES):
        b, _, _ = _shapes([(w, h)], 131, f32, seed=i)
        if i % 3 == 0:
            b.init[:, 2:] *= 2.0
        for side in {max(w, h), 32}:
            _equal(_fit(b, slots, max_side=side), _fit(b, 16, max_side=side, schedule=1))


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("slots", [32, 64])
def test_small_spots_of_any_shapes(slots, f32):
    shapes = [(w, h) for w in range(3, 9) for h in range(3, 9)]
    _, b, _ = _shapes(shapes, 11, f32)
    ref = _fit(b, 16)
    _equal(_fit(b, slots, max_side=8), ref)
    _equal(_fit(b, slots, schedule=1), ref)


@pytest.mark.parametrize("shapes", [[(30, 12)], [(12, 30)], [(20, 16), (29, 7)], [(4, 17), (16, 32)],
                                    [(30, 12), (12, 30)], [(32, 32), (5, 5)], [(3, 32), (3, 3)]])
@pytest.mark.parametrize("n", [1, 5, 203])
def test_a_few_wide_floats(shapes, n):
    """Spots end at different steps, so that a pass is left with the smaller ones."""
    _, b, _ = _shapes(shapes, -(-n // len(shapes)), True, seed=n)
    for schedule in (0, 1):
        _equal(_fit(b, 4, schedule=schedule), _fit(b, 16, schedule=schedule))
