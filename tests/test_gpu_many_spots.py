"""Start values of more spots than one launch takes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["moment_init", "peak_init"])
def test_more_spots_than_a_launch_has_threads_for(call):
    """A launch takes fewer than 2^32 threads, and the row kernels have one per spot.  The
    spots are unusable (no pixels are read) but for a few at the ends of the parts."""
    import torch

    import paper_2106_02045_amd as sf
    n = (1 << 32) + 131
    if torch.cuda.mem_get_info()[0] < 40 * n:
        pytest.skip("needs 40 bytes of GPU memory per spot")
    dev = "cuda:0"
    sizes = torch.zeros((n, 4), dtype=torch.uint8, device=dev)
    offsets = torch.zeros(n, dtype=torch.int64, device=dev)
    out = torch.zeros((n, 4), dtype=torch.float32, device=dev)
    data = torch.arange(25, dtype=torch.int32, device=dev).to(torch.uint16)
    at = [0, 1, (1 << 30) - 1, 1 << 30, (1 << 31) + 5, (1 << 32) - 1, 1 << 32, n - 1]
    for i in at:
        sizes[i, :2] = 5
    ctx = sf.Context(0)
    getattr(ctx, call)(data, sizes, offsets, out=out)
    torch.cuda.synchronize()
    want = getattr(ctx, call)(data, sizes[:1].clone(), offsets[:1].clone())[0]
    for i in at:
        assert torch.equal(out[i], want), i
    assert bool(torch.isfinite(want).all())
    for part in torch.split(out[:, 0], 1 << 28):
        out_nan = int(torch.isnan(part).sum())
        n -= out_nan
    assert n == len(at)
