"""Mixed precision: the position adjoint through the pair force (dl_dxy alone) is no further from
the FP64 call than the sum of the two parts, whose near sums meet the particle's own factors in
FP64 -- by leaf occupancy (target-centric units, both forms, mutual items), for smooth and random
circulations and cotangents.

Tolerance: both errors are root mean squares over at least 4096 rows; two of them scatter by 2%.
"""
import numpy as np
import pytest

from conftest import rel_l2
from test_gpu_sparse_units import OPT_DENSE_LEAF, _t

pytestmark = pytest.mark.gpu
OPT_NEAR_MUTUAL = 6


@pytest.mark.parametrize("leaf_sigma", [0.1, 1.0])
@pytest.mark.parametrize("per,dense", [(4, 32), (10, 32), (16, 32), (32, 32), (48, 32), (64, 32), (130, 32), (10, 1),
                                       (48, 1 << 30), (100, 0)],
                         ids=lambda v: str(v))  # dense 0: the mutual form off
def test_no_further_than_separate_sums(fmm_mod, per, dense, leaf_sigma):
    import torch
    depth = 5
    n, sigma, p = per << (2 * depth), leaf_sigma / (1 << depth), 16
    r = np.random.Generator(np.random.PCG64(per))
    xy = r.random((n, 2))
    tree = fmm_mod.Tree(_t(xy), depth, (0.0, 0.0, 1.0))
    if dense == 0:
        tree.set_option(OPT_NEAR_MUTUAL, 0)
    elif dense != 32:
        tree.set_option(OPT_DENSE_LEAF, dense)
    smooth = np.stack([np.sin(5 * xy[:, 0]), np.cos(3 * xy[:, 1])], axis=1)
    for g in (np.exp(-((xy - 0.5) ** 2).sum(axis=1) / 0.01), r.standard_normal(n)):
        for dl in (r.standard_normal((n, 2)), smooth):
            ref_g, ref_e, ref_s = (a.cpu().numpy() for a in tree.velocity_backward(_t(g), sigma, p, "fp64", _t(dl),
                                                                                  need_src=True))
            sep_g, sep_e, sep_s = (a.cpu().numpy() for a in tree.velocity_backward(_t(g), sigma, p, "mixed", _t(dl),
                                                                                  need_src=True))
            dg = torch.empty(n, dtype=torch.float64, device="cuda")
            dx = torch.empty(n, 2, dtype=torch.float64, device="cuda")
            tree.transport_vjp(_t(g), sigma, p, "mixed", _t(dl), 1.0, 0, dg, dx)
            assert rel_l2(dx.cpu().numpy(), ref_e + ref_s) <= 1.02 * rel_l2(sep_e + sep_s, ref_e + ref_s)
            assert rel_l2(dg.cpu().numpy(), ref_g) <= 1.02 * rel_l2(sep_g, ref_g)
