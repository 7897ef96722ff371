"""Brightest-pixel start values of spots with more columns than rows, which take the
lanes of their rows: the oracle's values, alone and beside spots of every other kind."""
import numpy as np
import pytest

import oracle
from test_gpu_init_sides import _batch, _up

pytestmark = pytest.mark.gpu

SHAPES = [(9, 8), (9, 3), (16, 8), (16, 3), (15, 9), (12, 5), (17, 8), (17, 16), (24, 3), (25, 8), (30, 12), (31, 16),
          (32, 3), (32, 9), (32, 16), (32, 17), (5, 5), (8, 32), (20, 20), (32, 32)]


@pytest.mark.parametrize("max_side", [16, 32])
def test_peak_values_by_rows(max_side):
    import paper_2106_02045_amd as sf
    ctx = sf.Context(0)
    shapes = [s for s in SHAPES if max(s) <= max_side]
    b = _batch(shapes, 61, seed=max_side)
    d, opts = _up(b.data), sf.default_options(max_side=max_side)
    want = oracle.peak_init_batch(b).astype(np.float32)
    np.testing.assert_array_equal(ctx.peak_init(d, _up(b.sizes), _up(b.offsets), opts).cpu().numpy(), want)
    for w, h in shapes:
        i = np.flatnonzero((b.sizes[:, 0] == w) & (b.sizes[:, 1] == h))
        alone = ctx.peak_init(d, _up(b.sizes[i]), _up(b.offsets[i]), opts)
        np.testing.assert_array_equal(alone.cpu().numpy(), want[i])
