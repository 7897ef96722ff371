"""Raw float spots with the latency hint: start values by a lane per column."""
import numpy as np
import pytest

import spotgen
from test_gpu_matrix import _shapes
from test_gpu_raw import _check_init, _run, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_side", [8, 16, 32])
@pytest.mark.parametrize("each", [1, 150])
def test_raw_floats_with_the_latency_hint(max_side, each):
    """Sides at the edges of the lanes, square and not, with negative pixels and unusable
    shapes: the oracle's estimate, and bit for bit the fit from the values reported."""
    import paper_2106_02045_amd as sf
    lo = {8: 3, 16: 9, 32: 17}[max_side]
    sides = (lo, lo + 2, max_side - 1, max_side)
    _, b, _ = _shapes([(w, h) for w in sides for h in (3,) + sides], each, True, seed=max_side)
    b = spotgen.SpotBatch(b.data - 150.0, b.sizes, b.offsets, b.init, b.truth, "f32")
    b.sizes[::17, 2] = 7
    opts = sf.default_options(max_side=max_side, plan_hint=sf.PLAN_LATENCY)
    raw, two, _ = _run(sf.Context(0), b, opts)
    _check_init(raw, b, opts, min_frac=0.999 if each > 1 else 0.9)
    for k in ("params", "chi2", "iters", "status", "evals"):
        assert _same(raw[k], two[k]), k
