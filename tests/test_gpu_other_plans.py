"""The mappings that a plan override (or the autotuner) chooses in place of the matrix-core
kernel: raw spots with the start values in the fit's own launch, and the latency hint,
which stays with the matrix-core kernel."""
import os

import numpy as np
import pytest

import spotgen
from parity import compare
from test_gpu_matrix import _equal, _shapes
from test_gpu_raw import _check_init, _run, _same

pytestmark = pytest.mark.gpu

# plan numbers by size class (<= 8, <= 16, <= 32 px): wide, wide without spills, narrow, lane-owned
GROUP_PLANS = ["0,2,4", "1,3,4", "1,9,10", "5,6,8", "5,7,8", "13,11,14", "13,12,15"]


def _ctx(**env):
    import paper_2106_02045_amd as sf
    os.environ.update(env)
    try:
        return sf.Context(0)
    finally:
        for k in env:
            del os.environ[k]


def _batch(max_side, f32):
    lo = {8: 3, 16: 9, 32: 17}[max_side]
    _, b, _ = _shapes([(w, h) for w in (lo, max_side) for h in (3, lo, max_side)], 40, f32, seed=max_side)
    b.sizes[::31, 2] = 5  # unusable
    return b


def _composition(ctx, b, opts):
    raw, two, _ = _run(ctx, b, opts)
    _check_init(raw, b, opts, min_frac=0.99)
    for k in ("params", "chi2", "iters", "status", "evals"):
        assert _same(raw[k], two[k]), k
    return raw


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("plans", GROUP_PLANS)
def test_raw_spots_with_other_plans(plans, f32):
    import paper_2106_02045_amd as sf
    ctx = _ctx(SPOTFIT_GROUP_PLAN=plans)
    for max_side in (8, 16, 32):
        b, opts = _batch(max_side, f32), sf.default_options(max_side=max_side)
        raw = _composition(ctx, b, opts)
        # the same decisions as the default plan from these start values
        b2 = spotgen.SpotBatch(b.data, b.sizes, b.offsets, raw["init"], b.truth, "raw")
        mine = _fit_default(b2, opts)
        same = (raw["status"] == mine["status"]) & (raw["iters"] == mine["iters"])
        assert same.mean() >= 0.99


def _fit_default(b, opts):
    import torch

    import paper_2106_02045_amd as sf
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    out = sf.Context(0).fit_spots(up(b.data), up(b.sizes), up(b.offsets), up(b.init), opts)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("plan", range(8))
def test_raw_spots_with_other_mixed_plans(plan, f32):
    import oracle
    import paper_2106_02045_amd as sf
    b = spotgen.workload("mixed_7to32", n=3000)
    if f32:
        b = spotgen.SpotBatch(b.data.astype(np.float32), b.sizes, b.offsets, b.init, b.truth, "f32")
    opts = sf.default_options(schedule=sf.SCHEDULE_MIXED)
    raw = _composition(_ctx(SPOTFIT_MIXED_PLAN=str(plan)), b, opts)
    b2 = spotgen.SpotBatch(b.data, b.sizes, b.offsets, raw["init"], b.truth, "raw")
    c = compare(raw, oracle.fit_batch(b2, oracle.default_opts(), threads=8), chi_band=1e-11, step_band=1e-9)
    assert c["strict_mismatch"] == 0 and c["tol_fail_same"] == 0


@pytest.mark.parametrize("schedule", [0, 1])
def test_the_latency_hint_stays_with_one_kernel(schedule):
    """Whatever plan an override keeps for throughput calls."""
    import torch

    import paper_2106_02045_amd as sf
    for max_side in (8, 16, 32):
        b = _batch(max_side, False)
        t = [torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in (b.data, b.sizes, b.offsets, b.init)]
        opts = sf.default_options(max_side=max_side, schedule=schedule, plan_hint=sf.PLAN_LATENCY)
        want = _fit_default(b, sf.default_options(max_side=max_side, schedule=schedule))
        for env in ({"SPOTFIT_GROUP_PLAN": "0,2,4"}, {"SPOTFIT_MIXED_PLAN": "0"}):
            got = _ctx(**env).fit_spots(*t, opts)
            torch.cuda.synchronize()
            _equal({k: v.cpu().numpy() for k, v in got.items()}, want)
