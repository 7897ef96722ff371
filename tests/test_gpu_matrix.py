"""The matrix-core fit kernel (the default plan) at the edges of its tiles.

A pass evaluates four spots in tiles of 4 x 4 pixels; a lane reads windows of 4
columns, cut off by the last row.  So every side from 3 to 32 is fitted, square
and not, alone in its batch (the build for one shape) and among others (the
build that goes over the largest spot's tiles), with 4, 16 and 64 spots per
wavefront, in order and through the sorted class lists.  A spot's sums depend on
its own shape alone: every one of these gives the same bits, and the oracle's
decisions.
"""
import os

import numpy as np
import pytest

import oracle
import spotgen
from parity import compare

pytestmark = pytest.mark.gpu


def _shapes(shapes, each, f32=False, seed=5):
    """`each` spots of every (w, h) of `shapes`, both models, cut from rendered
    images; start values from their moments."""
    rng = np.random.default_rng(seed)
    n = len(shapes) * each
    w = np.repeat([s[0] for s in shapes], each)
    h = np.repeat([s[1] for s in shapes], each)
    model = rng.integers(0, 2, n)
    off = rng.uniform(-0.4, 0.4, (n, 2))
    small = np.minimum(np.minimum(w, h), 12) / 6.0
    sig = rng.uniform(0.45, 0.9, (n, 2)) * small[:, None]
    sig[model == 0, 1] = sig[model == 0, 0]
    alpha, beta = 10.0 ** rng.uniform(2.5, 4, n), rng.uniform(10, 200, n)
    parts = spotgen._finish_chunk(rng, w, h, model, off, sig, alpha, beta, 2.0,
                                  np.float32 if f32 else np.uint16, spotgen.moment_init)
    b = spotgen._concat([parts], "shapes")
    order = rng.permutation(n)  # shapes of every size beside each other
    return b, b.subset(order), order


def _fit(b, slots=None, **kw):
    import torch

    import paper_2106_02045_amd as sf
    if slots:
        os.environ["SPOTFIT_MATRIX_SLOTS"] = str(slots)
    try:
        ctx = sf.Context(0)
    finally:
        os.environ.pop("SPOTFIT_MATRIX_SLOTS", None)
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    out = ctx.fit_spots(up(b.data), up(b.sizes), up(b.offsets), up(b.init), sf.default_options(**kw),
                        want_evals=True)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


def _equal(a, b):
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


SQUARE = [(s, s) for s in range(3, 33)]
UNEVEN = [(3, 32), (32, 3), (4, 5), (5, 4), (3, 4), (4, 3), (8, 9), (9, 8), (12, 13), (16, 17),
          (17, 16), (20, 21), (31, 7), (7, 31), (29, 32), (32, 29), (15, 3), (3, 16)]


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("shapes", [SQUARE, UNEVEN], ids=["square", "uneven"])
def test_every_shape_in_any_company(shapes, f32):
    apart, among, order = _shapes(shapes, 37, f32)
    mixed = {s: _fit(among, s, schedule=1) for s in (4, 16, 64)}
    _equal(mixed[4], mixed[16])
    _equal(mixed[4], mixed[64])
    _equal(mixed[4], _fit(among, 16))  # uniform schedule
    # each shape as a batch of its own
    back = np.argsort(order)
    npx = 37
    for i, (w, h) in enumerate(shapes):
        one = apart.subset(np.arange(i * npx, (i + 1) * npx))
        got = _fit(one, (4, 16, 64)[i % 3], max_side=max(w, h))
        _equal(got, {k: v[back[i * npx:(i + 1) * npx]] for k, v in mixed[4].items()})
    r = oracle.fit_batch(among, oracle.default_opts(), threads=8)
    c = compare(mixed[4], r, chi_band=1e-11, step_band=1e-9)
    assert c["strict_mismatch"] == 0 and c["tol_fail_same"] == 0


@pytest.mark.parametrize("f32", [False, True])
def test_more_spots_than_the_chip_holds(f32):
    """Batches that draw from the spot counters (several rounds), with a ragged
    end, in order and through the sorted lists (above 65,536 spots), give the
    bits of the same spots in one round."""
    b = spotgen.workload("mixed_7to32", n=70003, threads=8)
    if f32:
        b = spotgen.SpotBatch(b.data.astype(np.float32), b.sizes, b.offsets, b.init, b.truth, "f32")
    ref = _fit(b, 64)                       # one round, in order
    _equal(ref, _fit(b, 4, schedule=1))     # sorted lists, many rounds
    _equal(ref, _fit(b, 16, schedule=1))
    _equal(ref, _fit(b, 4))                 # in order, many rounds


def test_retries_evaluate_the_best_point_again():
    """Spots whose trials are often worse: a wavefront of 64 spots re-evaluates
    the best point for a retry instead of keeping its normal equations (as with
    4 and 16), and nothing of it shows: evaluation counts, steps, results."""
    b = spotgen.workload("mixed_low_contrast", n=6000)
    b.init[:, 2:] *= 2.5  # far starts: many retries with more damping
    a, c, d = (_fit(b, s, schedule=1) for s in (4, 16, 64))
    assert (a["evals"][:, 1] > a["iters"]).sum() > 50
    _equal(a, c)
    _equal(a, d)
    r = oracle.fit_batch(b, oracle.default_opts(), threads=8)
    k = compare(a, r, chi_band=1e-11, step_band=1e-9)
    assert k["strict_mismatch"] == 0


@pytest.mark.parametrize("n", [12289, 40001, 262200])
def test_batch_sizes_of_every_build(n):
    """Batches that take 16, 32 and 64 spots per wavefront by themselves, the last
    of them through the sorted class lists: the bits of the same spots in a small
    batch.  Every spot is in the batch several times, on one copy of its pixels."""
    _, b, _ = _shapes([(3, 4), (4, 4), (7, 7), (8, 9), (9, 9), (12, 17), (25, 17)], 121)
    m = b.sizes.shape[0]
    t = np.arange(n) % m
    big = spotgen.SpotBatch(b.data, b.sizes[t], b.offsets[t], b.init[t], b.truth, "tiled")
    ref = _fit(b, 4, schedule=1)
    _equal(_fit(big, schedule=1), {k: v[t] for k, v in ref.items()})


@pytest.mark.parametrize("n", [1, 3, 256, 257, 512, 513, 1025])
def test_small_mixed_batches_spread_over_the_chip(n):
    """One, two and four spots per wavefront of the build for four (the last
    wavefront part full): the bits of the same spots in one larger batch."""
    _, b, _ = _shapes([(5, 7), (9, 9), (17, 12), (24, 31)], 300)
    ref = _fit(b, 16, schedule=1)
    _equal(_fit(b.subset(np.arange(n)), schedule=1), {k: v[:n] for k, v in ref.items()})
