"""Served frames with and without their size-class lists."""
import os

import numpy as np
import pytest

import spotgen

pytestmark = pytest.mark.gpu


def _frame(n, side=9):
    b = spotgen.workload("small_11x11", n=n)
    b.sizes[:, :2] = side
    px = np.concatenate([b.data[o:o + side * side] for o in b.offsets])
    return px, b.sizes, b.init


def _serve(frame, budget, **env):
    import paper_2106_02045_amd as sf
    os.environ.update(env)
    try:
        sv = sf.Server(0, sf.default_options(schedule=sf.SCHEDULE_MIXED), device_mem_budget=budget)
    finally:
        for k in env:
            del os.environ[k]
    try:
        got = sv.submit(*frame)
        return None if got is None else sv.wait(got[0])
    finally:
        sv.close()


def test_a_frame_brings_no_lists_that_nothing_reads():
    """623,700 bytes of pixels and 32 of records a spot fit the pixel ring of a 1 MiB budget,
    with 12 more a spot for the lists they do not; a mapping that reads them needs the room."""
    frame = _frame(3850)
    small = _serve(frame, 1 << 20)
    assert small is not None
    assert _serve(frame, 1 << 20, SPOTFIT_MIXED_PLAN="7") is None
    large = _serve(frame, 1 << 24)
    for k in large:
        np.testing.assert_array_equal(small[k], large[k])
    other = _serve(frame, 1 << 24, SPOTFIT_MIXED_PLAN="7")
    np.testing.assert_array_equal(other["status"], large["status"])
    np.testing.assert_array_equal(other["iters"], large["iters"])
