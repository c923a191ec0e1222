"""What destroyed uniform trees leave reserved on the device is bounded, also beside a tree that
lives on and keeps the runtime's pool in use.
"""
import pytest

pytestmark = pytest.mark.gpu
IDLE_BYTES = 1 << 30  # kIdleBytes


def test_pool_beside_a_living_tree(fmm_mod):
    import torch
    n = 1 << 26  # arrays of some 3 GiB a tree
    xy = torch.rand(n, 2, dtype=torch.float64, device="cuda")
    box = (0.0, 0.0, 1.0)
    first = fmm_mod.Tree(xy, 10, box)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    second = fmm_mod.Tree(xy, 10, box)
    torch.cuda.synchronize()
    arrays = before - torch.cuda.mem_get_info()[0]
    second.close()
    held = before - torch.cuda.mem_get_info()[0]
    first.close()
    assert arrays > 40 * n  # the arrays of fixed size alone
    assert held <= IDLE_BYTES + (64 << 20), held
