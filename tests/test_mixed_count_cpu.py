"""Mixed-schedule batches of 2^31 spots and more are refused on the host before
anything is launched, with either hint and by every call that takes one."""
import ctypes

import pytest

import paper_2106_02045_amd as sf


@pytest.mark.parametrize("hint", [sf.PLAN_THROUGHPUT, sf.PLAN_LATENCY])
@pytest.mark.parametrize("n", [1 << 31, 1 << 40])
def test_too_many_mixed_spots_are_refused(n, hint):
    # a zeroed block as context and addresses that are not looked at: on a machine
    # without a GPU a call that gets past the check ends with a HIP error instead
    L, ctx = sf.lib(), ctypes.create_string_buffer(4096)
    fake = ctypes.cast(ctx, ctypes.c_void_p)
    o = sf.default_options(schedule=sf.SCHEDULE_MIXED, plan_hint=hint)
    opt = ctypes.byref(o)
    rep = sf.TuneReport()
    assert L.spotfit_fit_spots(fake, 1, 0, 1, 1, 1, n, opt, 1, 1, 1, 1, None, None) == -2
    assert b"2^31" in L.spotfit_last_error()
    assert L.spotfit_fit_raw(fake, 1, 0, 1, 1, n, opt, 1, 1, 1, 1, 1, None, None) == -2
    assert L.spotfit_autotune(fake, 1, 0, 1, 1, 1, n, opt, 1, 1, 1, 1, 3, ctypes.byref(rep), None) == -2
    assert L.spotfit_fit_spots_noalloc(fake, 1, 0, 1, 1, 1, n, opt, 1, 1, 1, 1, None, None) == -2
