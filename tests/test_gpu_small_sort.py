"""Sorts of one workgroup: the device build against the host build at the sizes where rounds,
wavefronts and the sort itself change, for an even and an odd number of passes.  Positions on a
coarse grid make many equal keys, whose particles must keep their order.  Whole numbers: exact.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
SIZES = [2, 63, 64, 65, 1023, 1024, 1025, 2049, 4096, 4097, 7169, 8191, 8192, 8193]


@pytest.mark.parametrize("depth", [2, 4])  # 16 and 20 bits of key
@pytest.mark.parametrize("n", SIZES)
def test_permutation(fmm_mod, n, depth):
    import torch
    r = np.random.Generator(np.random.PCG64(n))
    xy = torch.from_numpy(r.integers(0, 90, (n, 2)) / 90.0).to("cuda")
    box = (0.0, 0.0, 1.0)
    td = fmm_mod.Tree(xy, depth, box, builder="device")
    th = fmm_mod.Tree(xy, depth, box, builder="host")
    assert td.info() == th.info() and td.near_plan() == th.near_plan()
    for a, b in zip(td.permutation(), th.permutation()):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
