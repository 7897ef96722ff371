"""One spot, one result: whatever batch, schedule, hint, largest side or number of spots per
wavefront, also for spots whose fit hangs on the last bit (images without a spot, far
starts, nearly singular normal equations, pixels that are not finite)."""
import os

import numpy as np
import pytest

import spotgen

pytestmark = pytest.mark.gpu


def _hard(f32, max_side, seed):
    """Spots of every kind of shape; noise, constant images and lone pixels beside
    Gaussians, start values up to 2.5 sigmas off and some unusable ones."""
    rng = np.random.default_rng(seed)
    n = 1500
    wh = rng.integers(3, max_side + 1, (40, 2))[rng.integers(0, 40, n)]
    wh[: n // 3] = rng.integers(3, min(max_side, 7) + 1, (n // 3, 2))
    npx = wh[:, 0] * wh[:, 1]
    offsets = np.cumsum(npx) - npx + np.arange(n) % 3
    data = np.zeros(int(offsets[-1] + npx[-1]))
    init = np.zeros((n, 4), np.float32)
    for i, (w, h) in enumerate(wh):
        x0, y0 = (w - 1) / 2 + rng.uniform(-0.6, 0.6), (h - 1) / 2 + rng.uniform(-0.6, 0.6)
        s = min(w, h) / 6 * rng.uniform(0.5, 1.4)
        y, x = np.mgrid[:h, :w]
        g = 10 ** rng.uniform(1, 4.5) * np.exp(-0.5 * ((x - x0) ** 2 + (y - y0) ** 2) / s**2) + rng.uniform(0, 300)
        g = rng.poisson(np.minimum(g, 60000)).astype(np.float64).ravel()
        kind = rng.random()
        if kind < 0.05:
            g[:] = rng.choice([0, 1, 65535])
        elif kind < 0.1:
            g = rng.integers(0, 50, w * h).astype(np.float64)
        elif f32 and kind < 0.15:
            g[rng.integers(0, w * h)] = rng.choice([np.nan, np.inf, -np.inf, 1e38, -3e38, 1e-40])
        data[offsets[i]:offsets[i] + w * h] = g
        init[i] = (x0 + rng.normal(0, 0.5), y0 + rng.normal(0, 0.5), s * rng.uniform(0.5, 2.5), s * rng.uniform(0.5, 2.5))
    bad = rng.random(n) < 0.02
    init[bad, rng.integers(0, 4)] = rng.choice([np.nan, np.inf, -1, 1e30, 1e-30])
    sizes = np.zeros((n, 4), np.uint8)
    sizes[:, :2], sizes[:, 2] = wh, rng.integers(0, 2, n)
    data = data.astype(np.float32) if f32 else np.clip(data, 0, 65535).astype(np.uint16)
    return spotgen.SpotBatch(data, sizes, offsets.astype(np.int64), init, None, "hard")


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("max_side", [8, 16, 32])
def test_same_bits_in_every_build(max_side, f32):
    import torch

    import paper_2106_02045_amd as sf
    b = _hard(f32, max_side, 10 * max_side + f32)
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    d = [up(x) for x in (b.data, b.sizes, b.offsets, b.init)]
    ctx = {}
    for slots in (4, 16, 32, 64):
        os.environ["SPOTFIT_MATRIX_SLOTS"] = str(slots)
        ctx[slots] = sf.Context(0)
        del os.environ["SPOTFIT_MATRIX_SLOTS"]

    def fit(slots, idx=slice(None), **kw):
        out = ctx[slots].fit_spots(d[0], *(t[idx].contiguous() for t in d[1:]), sf.default_options(**kw), want_evals=True)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in out.items()}

    want = fit(4, max_side=max_side)
    assert len(np.unique(want["status"])) >= 4
    for slots in ctx:
        for kw in (dict(max_side=max_side), dict(), dict(schedule=1), dict(plan_hint=1)):
            got = fit(slots, **kw)
            for k in want:
                np.testing.assert_array_equal(got[k], want[k], err_msg=f"{k}, {slots} slots, {kw}")
    order = np.random.default_rng(0).permutation(b.n)[:700]
    got = fit(64, torch.from_numpy(order).to("cuda:0"))
    for k in want:
        np.testing.assert_array_equal(got[k], want[k][order], err_msg=f"{k}, in other company")
