"""Target-centric units over sparse leaves: the source leaves of a unit staged together, at
the leaf sizes where the lane mapping, the batches of 64 sources and the partial sums change,
forward and adjoint, both trees, against the oracle.

Tolerances: the repository's gates for the near field (FP64 1e-12 of ragged leaves, mixed
1e-5) and for the gradients (FP64 1e-9, mixed 1e-4).
"""
import numpy as np
import pytest

from conftest import rel_l2

pytestmark = pytest.mark.gpu
BOX = (0.0, 0.0, 1.0)
OPT_DENSE_LEAF = 7
FWD = {"fp64": 1e-12, "mixed": 1e-5}
BWD = {"fp64": 1e-9, "mixed": 1e-4}


def _t(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def _leaves(sizes, depth, seed):
    """Leaf k of the given sizes filled with that many points, row by row over the grid."""
    r = np.random.Generator(np.random.PCG64(seed))
    side = 1 << depth
    xy = [(np.array([k % side, k // side]) + r.random((m, 2))) / side for k, m in enumerate(sizes)]
    xy = np.concatenate(xy)
    return xy[r.permutation(len(xy))], r.standard_normal(len(xy)), r


SIZES = [1, 64, 0, 9, 17, 2, 8, 33, 10, 12, 13, 63, 16, 15, 21, 22, 31, 32, 3, 5, 24, 65, 7, 40, 4, 64, 11, 6, 20, 1, 48, 14]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes", [[s for s in SIZES if s <= 64], SIZES, [1] * 64, [64] * 40, [0, 0, 5]],
                         ids=["ragged", "ragged65", "ones", "full", "corner"])
def test_uniform_units(fmm_mod, oracle_mod, sizes, precision):
    depth = 3
    xy, g, r = _leaves(sizes, depth, 5)
    dl = r.standard_normal(xy.shape)
    for sigma in (0.1, 0.008):  # every pair with the exponential; part of the leaves beyond it
        tree = fmm_mod.Tree(_t(xy), depth, BOX)
        on = oracle_mod.fmm_velocity(xy, g, sigma, depth, 6, BOX, parts=True)[0]
        refs = oracle_mod.fmm_grad_full(xy, g, sigma, depth, 6, dl, BOX)
        for dense in (32, 1 << 30):
            tree.set_option(OPT_DENSE_LEAF, dense)
            near = tree.velocity_parts(_t(g), sigma, 6, precision)[0].cpu().numpy()
            assert rel_l2(near, on) < FWD[precision], (sigma, dense)
        for need_src in (False, True):
            got = tree.velocity_backward(_t(g), sigma, 6, precision, _t(dl), need_src=need_src)
            for name, a, b in zip(("dgamma", "dx_eval", "dx_src"), got, refs):
                assert rel_l2(a.cpu().numpy(), b) < BWD[precision], (sigma, name)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("max_leaf", [3, 20, 64, 80])
def test_adaptive_units(fmm_mod, oracle_mod, max_leaf, precision):
    """A coarse leaf beside a line of points split down to the deepest level: with max_leaf 3
    its list of adjacent leaves is longer than a wavefront."""
    r = np.random.Generator(np.random.PCG64(max_leaf))
    line = np.stack([0.5 + 0.002 * r.random(1500), 0.25 + 0.25 * r.random(1500)], axis=1)
    xy = np.concatenate([line, 0.05 + 0.4 * r.random((max_leaf, 2)) * [1, 0.5] + [0, 0.25], r.random((60, 2))])
    g, dl = r.standard_normal(len(xy)), r.standard_normal(xy.shape)
    depth, p = 9, 8
    tree = fmm_mod.ATree(_t(xy), max_leaf, depth, BOX)
    for sigma in (0.002, 0.0002):
        ref = oracle_mod.afmm_velocity(xy, g, sigma, max_leaf, depth, p, BOX)
        uv = tree.velocity(_t(g), sigma, p, precision).cpu().numpy()
        assert rel_l2(uv, ref) < (1e-11 if precision == "fp64" else 1e-5), sigma
        refs = oracle_mod.afmm_grad(xy, g, sigma, max_leaf, depth, p, dl, BOX)
        got = tree.velocity_backward(_t(g), sigma, p, precision, _t(dl), need_src=True)
        for name, a, b in zip(("dgamma", "dx_eval", "dx_src"), got, refs):
            assert rel_l2(a.cpu().numpy(), b) < BWD[precision], (sigma, name)
