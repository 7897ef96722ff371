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
