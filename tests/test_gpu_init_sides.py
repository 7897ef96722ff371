"""Start values of spots that are smaller than the launch is for: the values do not
depend on the largest side that is allowed nor on the spots beside one, and small spots do
not pay for the lanes that large ones would take."""
import time

import numpy as np
import pytest

import spotgen

pytestmark = pytest.mark.gpu


def _batch(shapes, each, seed=2):
    """`each` spots of every (w, h), noise on a slope (every start value its own), in random order."""
    rng = np.random.default_rng(seed)
    wh = rng.permutation(np.repeat(shapes, each, axis=0))
    n = len(wh)
    px = wh[:, 0] * wh[:, 1]
    offsets = np.cumsum(px) - px + np.arange(n) % 3  # odd addresses too
    data = rng.integers(0, 65536, int(offsets[-1] + px[-1])).astype(np.uint16)
    sizes = np.zeros((n, 4), np.uint8)
    sizes[:, :2], sizes[:, 2] = wh, rng.integers(0, 2, n)
    return spotgen.SpotBatch(data, sizes, offsets.astype(np.int64), np.zeros((n, 4), np.float32), None, "noise")


def _up(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


@pytest.mark.parametrize("call", ["moment_init", "peak_init"])
def test_values_do_not_depend_on_the_launch(call):
    """Sides at the edges of the 8, 16 and 32 lanes and of the windows of 4 columns, with
    unusable spots among them: together under the default options, and by shape under
    the smallest options that take it."""
    import torch

    import paper_2106_02045_amd as sf
    ctx = sf.Context(0)
    shapes = [(3, 3), (8, 8), (3, 8), (9, 9), (8, 9), (9, 3), (16, 16), (5, 16), (17, 17), (3, 17), (17, 3),
              (20, 32), (21, 20), (24, 24), (25, 30), (28, 17), (29, 32), (32, 32), (32, 5)]
    b = _batch(shapes, 67)
    bad = np.arange(b.n) % 11 == 3
    b.sizes[bad, 2] = 9
    d, o = _up(b.data), _up(b.offsets)
    got = getattr(ctx, call)(d, _up(b.sizes), o).cpu().numpy()
    assert np.isnan(got[bad]).all() and np.isfinite(got[~bad]).all()
    for w, h in shapes:
        i = np.flatnonzero((b.sizes[:, 0] == w) & (b.sizes[:, 1] == h))
        alone = getattr(ctx, call)(d, _up(b.sizes[i]), _up(b.offsets[i]), sf.default_options(max_side=max(w, h)))
        np.testing.assert_array_equal(alone.cpu().numpy(), got[i])
    torch.cuda.synchronize()


@pytest.mark.parametrize("call", ["moment_init", "peak_init"])
@pytest.mark.parametrize("side", [7, 9])
def test_small_spots_under_the_default_options(call, side):
    """Sides up to 32 allowed, spots of 7 or 9 px: with 32 lanes for each of them the
    launch took 3 to 5 times as long as with their own largest side; half as much again
    and a launch's noise are allowed for."""
    import torch

    import paper_2106_02045_amd as sf
    ctx = sf.Context(0)
    b = _batch([(side, side)], 200000)
    d = (_up(b.data), _up(b.sizes), _up(b.offsets))
    out = torch.empty((b.n, 4), dtype=torch.float32, device="cuda:0")

    def us(opts):
        best = 1e9
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                getattr(ctx, call)(*d, opts, out=out)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) / 10)
        return best * 1e6

    own, wide = us(sf.default_options(max_side=side)), us(None)
    own, wide = min(own, us(sf.default_options(max_side=side))), min(wide, us(None))
    print(f"own side {own:.1f} us, default options {wide:.1f} us")
    assert wide <= 1.5 * own + 5.0
