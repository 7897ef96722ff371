"""Mixed batches large enough for the sorted class lists (above 262,144 spots): every build
of the matrix-core kernel, both pixel types and every workspace the lists can be in,
against the bits of the same spots in a small batch in order."""

import numpy as np
import pytest

import spotgen
from test_gpu_matrix import _equal, _fit, _shapes

pytestmark = pytest.mark.gpu

N = 262144 + 61  # a ragged end


def _tiled(f32, n=N):
    """Every spot many times, on one copy of its pixels; all classes, some unusable."""
    shapes = [(3, 4), (7, 7), (8, 8), (9, 5), (12, 17), (16, 16), (25, 17), (32, 30)]
    _, b, _ = _shapes(shapes, 97, f32)
    b.sizes[::41, 2] = 4
    t = np.random.default_rng(n).integers(0, b.n, n)
    return b, spotgen.SpotBatch(b.data, b.sizes[t], b.offsets[t], b.init[t], b.truth, "tiled"), t


def _up(b):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in (b.data, b.sizes, b.offsets, b.init)]


def _host(out):
    import torch
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


def _take(ref, t, keys=None):
    return {k: v[t] for k, v in ref.items() if keys is None or k in keys}


@pytest.mark.parametrize("f32", [False, True])
def test_lists_in_every_build(f32):
    small, big, t = _tiled(f32)
    want = _take(_fit(small, 16), t)
    for slots in (None, 4, 16, 32, 64):
        _equal(_fit(big, slots, schedule=1), want)


@pytest.mark.parametrize("f32", [False, True])
def test_lists_in_the_fixed_scratch_memory(f32):
    """A large call, then a smaller one that still takes the lists: nothing of the first
    one's counters or lists shows."""
    import paper_2106_02045_amd as sf
    ctx, opts = sf.Context(0), sf.default_options(schedule=1)
    for n in (sf.NOALLOC_MAX_SPOTS, N, 5000):
        small, big, t = _tiled(f32, n)
        want = _take(_fit(small, 16), t)
        _equal(_host(ctx.fit_spots_noalloc(*_up(big), opts, want_evals=True)), want)


@pytest.mark.parametrize("raw", [False, True])
def test_lists_in_a_captured_fit(raw):
    """The graph's own workspace: replays are not touched by a larger call on the context,
    which makes its workspace grow, nor that by them."""
    import torch

    import paper_2106_02045_amd as sf
    small, big, t = _tiled(False)
    ctx, opts = sf.Context(0), sf.default_options(schedule=1)
    d = _up(big)
    keys = ("params", "chi2", "iters", "status")
    if raw:
        s = _up(small)
        want = _take(_host(ctx.fit_raw(*s[:3], opts)), t, keys)
    else:
        want = _take(_fit(small, 16), t, keys)
    g = ctx.graph(d[0], d[1], d[2], None if raw else d[3], opts)
    small2, big2, t2 = _tiled(True, 2 * N)
    d2, want2 = _up(big2), _take(_fit(small2, 16), t2, keys)
    for _ in range(3):
        for v in g.out.values():
            v.zero_()
        g.launch()
        torch.cuda.synchronize()
        _equal({k: g.out[k].cpu().numpy() for k in keys}, want)
        got = _host(ctx.fit_spots(*d2, opts))
        _equal({k: got[k] for k in keys}, want2)


def test_lists_of_a_context_after_larger_ones():
    import paper_2106_02045_amd as sf
    ctx, opts = sf.Context(0), sf.default_options(schedule=1)
    for n in (3 * N, N, 4000, N + 1):
        small, big, t = _tiled(False, n)
        _equal(_host(ctx.fit_spots(*_up(big), opts, want_evals=True)), _take(_fit(small, 16), t))


def test_lists_of_a_served_frame():
    """One frame of that many spots brings its class lists along."""
    import paper_2106_02045_amd as sf
    n = N
    small, big, t = _tiled(False, n)
    shapes = big.sizes[:, 0].astype(np.int64) * big.sizes[:, 1]
    pixels = np.concatenate([small.data[o:o + p] for o, p in zip(big.offsets, shapes)])
    want = _take(_fit(small, 16), t, ("params", "chi2", "iters", "status"))
    sv = sf.Server(0, sf.default_options(schedule=1), device_mem_budget=1 << 30)
    try:
        for _ in range(2):
            ticket, out = sv.submit(pixels, big.sizes, big.init)
            got = sv.wait(ticket)
            _equal({k: np.asarray(got[k]) for k in want}, want)
    finally:
        sv.close()
