"""What the autotuner times and what it keeps."""
import numpy as np
import pytest

import spotgen

pytestmark = pytest.mark.gpu


def _on_gpu(b):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in (b.data, b.sizes, b.offsets, b.init)]


@pytest.mark.parametrize("schedule", [0, 1])
def test_latency_tuning_leaves_the_throughput_plan(schedule):
    """Every call with the latency hint runs the same kernel, so there is one candidate;
    what throughput calls of the context take afterwards is what they took before."""
    import torch

    import paper_2106_02045_amd as sf
    b = spotgen.workload("mixed_7to32", n=3000) if schedule else spotgen.config(0, n=3000)
    t = _on_gpu(b)
    side = int(b.sizes[:, :2].max())
    latency = sf.default_options(max_side=side, schedule=schedule, plan_hint=sf.PLAN_LATENCY)
    throughput = sf.default_options(max_side=side, schedule=schedule)
    want = sf.Context(0).fit_spots(*t, throughput)
    ctx = sf.Context(0)
    out, rep = ctx.autotune(*t, latency, reps=1)
    assert len(rep["plan_id"]) == 1 and rep["chosen_plan"] == rep["plan_id"][0]
    got = ctx.fit_spots(*t, throughput)
    torch.cuda.synchronize()
    for k in want:
        np.testing.assert_array_equal(got[k].cpu().numpy(), want[k].cpu().numpy())
        np.testing.assert_array_equal(out[k].cpu().numpy(), want[k].cpu().numpy())


def test_no_plan_is_left_untimed():
    """Spots of at most 8 px fit every lane mapping, 17 with the matrix-core kernel's,
    and the report holds the 16 fastest: the slowest of a batch that fills the GPU is
    the mapping with 32 lanes per spot, so that all the others are reported."""
    import paper_2106_02045_amd as sf
    b = spotgen.workload("small_11x11", n=4000)
    t = np.arange(300000) % b.n
    rng = np.random.default_rng(1)
    sizes, offsets, init = b.sizes[t], b.offsets[t], b.init[t]
    sizes[:, :2] = 7  # 7 x 7 pixels of each spot's 121, wherever they start
    init[:, :2] = rng.uniform(2.5, 3.5, (len(t), 2))
    b = spotgen.SpotBatch(b.data, sizes, offsets, init, b.truth, "7x7")
    ctx = sf.Context(0)
    _, rep = ctx.autotune(*_on_gpu(b), sf.default_options(max_side=8), reps=2)
    print(dict(zip(rep["plan_id"], rep["plan_ms"])))
    assert len(rep["plan_id"]) == 16 and len(set(rep["plan_id"])) == 16
    assert rep["chosen_plan"] == rep["plan_id"][int(np.argmin(rep["plan_ms"]))]
    assert 15 in rep["plan_id"] and 16 in rep["plan_id"]  # the last mapping, and the matrix-core kernel
