"""Stop reasons, iteration counts and evaluation totals of a fitted batch, at the
edges of the blocks that count them, against numpy: whole numbers, exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_evals", [True, False])
@pytest.mark.parametrize("n", [1, 63, 65, 1025, 4096, 4097, 100003, 128 * 4096, 128 * 4096 + 1, 1500007])
def test_counts_match_numpy(n, with_evals):
    import torch

    import paper_2106_02045_amd as sf
    rng = np.random.default_rng(n)
    out = {"status": rng.integers(-1, 8, n).astype(np.int32),  # values that are no status too
           "iters": rng.integers(-3, 100, n).astype(np.int32)}
    if with_evals:
        out["evals"] = rng.integers(-2, 2**31 - 1, (n, 2)).astype(np.int32)
    ctx = sf.Context(0)
    dev = {k: torch.from_numpy(v).to("cuda:0") for k, v in out.items()}
    for _ in range(2):  # nothing is left over from a call
        st = ctx.stats(dev)
        assert st["n_spots"] == n
        s = out["status"]
        np.testing.assert_array_equal(st["status_count"], [(s == k).sum() for k in range(6)])
        np.testing.assert_array_equal(st["iters_hist"],
                                      np.bincount(np.clip(out["iters"], 0, 64), minlength=65))
        for i, k in enumerate(("grad_evals", "trial_evals")):
            want = int(np.maximum(out["evals"][:, i].astype(np.int64), 0).sum()) if with_evals else 0
            assert st[k] == want


def test_contexts_take_turns():
    """Every context has its own counts, whether it is the first call on it or not, and
    one that never counted is destroyed like the others."""
    import torch

    import paper_2106_02045_amd as sf
    dev = [{"status": torch.full((k + 1,), k, dtype=torch.int32, device="cuda:0"),
            "iters": torch.full((k + 1,), 10 * k, dtype=torch.int32, device="cuda:0")} for k in range(3)]
    ctx = [sf.Context(0) for _ in range(4)]
    for _ in range(2):
        for k in range(3):
            st = ctx[k].stats(dev[k])
            assert st["n_spots"] == k + 1 and st["status_count"][k] == k + 1 and st["iters_hist"][10 * k] == k + 1
    for c in ctx:
        c.close()
