"""Host copies of a captured fit at the edges of the kernel that makes the small
ones (8 bytes per thread; other alignments and last bytes by themselves; above
1 MiB in all the copy engine): the device has the host's bytes after every replay,
and the host the results of a direct fit."""
import numpy as np
import pytest

import spotgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("skip", [0, 1, 2])  # elements before the pixels: their alignment
@pytest.mark.parametrize("extra", [0, 1, 2, 3, 524288 - 4 * 169 - 16 * 4 // 2, 524288, 700001])
def test_bytes_of_every_alignment(extra, skip):
    import torch

    import paper_2106_02045_amd as sf
    _, _, frames = spotgen.drift_frames(3, n_markers=4, side=13, seed=7)
    ctx = sf.Context(0)
    opts = sf.default_options(max_side=13)
    up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    f0 = frames[0]
    npx = f0.data.size
    data = torch.zeros(npx + extra + skip, dtype=torch.uint16, device="cuda:0")[skip:]
    init = up(f0.init)
    out = {k: torch.empty((4, 6) if k == "params" else 4, device="cuda:0",
                          dtype=torch.int32 if k in ("iters", "status") else torch.float32)
           for k in ("params", "chi2", "iters", "status")}
    host = {k: torch.empty(v.numel() + 1, dtype=v.dtype).pin_memory()[skip % 2:][:v.numel()].view(v.shape)
            for k, v in out.items()}
    host["data"] = torch.empty(npx + extra + skip, dtype=torch.uint16).pin_memory()[skip:]
    host["init"] = torch.empty((4, 4), dtype=torch.float32).pin_memory()
    g = ctx.graph(data, up(f0.sizes), up(f0.offsets), init, opts, out=out, host=host)
    rng = np.random.default_rng(extra)
    for f in frames + frames[:1]:
        px = rng.integers(0, 65536, npx + extra).astype(np.uint16)
        px[:npx] = f.data
        host["data"].copy_(torch.from_numpy(px))
        host["init"].copy_(torch.from_numpy(f.init))
        for k in out:
            host[k].fill_(-1)
        float((torch.arange(100000, device="cuda:0", dtype=torch.float32) * 0.5).sum().item())
        g.launch()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(data.cpu().numpy(), px)
        want = ctx.fit_spots(up(f.data), up(f.sizes), up(f.offsets), up(f.init), opts)
        torch.cuda.synchronize()
        for k in out:
            np.testing.assert_array_equal(host[k].numpy(), want[k].cpu().numpy())
    g.close()
