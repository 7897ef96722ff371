"""Which host arrays the copy kernel takes: those that lie in one pinned allocation
(anything else stays with the copy engine).  Addresses are looked up, not read."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


def test_only_one_pinned_allocation():
    import torch

    import paper_2106_02045_amd as sf
    look = sf.lib()["_ZN2sf14pinned_addressEPKvl"]
    look.restype, look.argtypes = ctypes.c_void_p, [ctypes.c_void_p, ctypes.c_int64]
    torch.zeros(1, device="cuda:0")
    a, b = (torch.empty(1 << 16, dtype=torch.uint8).pin_memory() for _ in range(2))
    a, b = sorted((a, b), key=lambda t: t.data_ptr())
    p, n = a.data_ptr(), a.numel()
    assert look(p, n) is not None
    assert look(p + 7, 1) == look(p, 1) + 7 and look(p + n - 1, 1) is not None
    # from one allocation into another, both ends pinned
    assert look(p + n - 16, b.data_ptr() + 16 - (p + n - 16)) is None
    assert look(p + 1, n * 1024) is None      # past the allocation's end
    assert look(torch.empty(4096, dtype=torch.uint8).data_ptr(), 64) is None  # pageable
    assert look(torch.empty(64, device="cuda:0").data_ptr(), 64) is None      # device memory
