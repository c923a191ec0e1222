"""Leaves of the adaptive tree that the depth limit leaves with thousands of particles: their mutual
items run over many tiles (one wavefront's chain each), forward and adjoint, against the oracle.

Tolerances: the repository's gates for the velocities (FP64 1e-10, mixed 1e-5) and for the
gradients (FP64 1e-9, mixed 1e-4).
"""
import numpy as np
import pytest

from conftest import rel_l2
from test_gpu_pair_force import _check
from test_gpu_sparse_units import BOX, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_leaves_at_the_depth_limit(fmm_mod, oracle_mod, precision):
    r = np.random.Generator(np.random.PCG64(31))
    depth, max_leaf, p, sigma = 4, 30, 8, 0.004
    # two neighbouring finest cells of 1900 and 700 particles, one of 65, and a background
    cells = [((5, 9), 1900), ((6, 9), 700), ((6, 10), 65)]
    xy = np.concatenate([(np.array(c) + r.random((m, 2))) / (1 << depth) for c, m in cells] + [r.random((600, 2))])
    xy = xy[r.permutation(len(xy))]
    g, dl = r.standard_normal(len(xy)), r.standard_normal(xy.shape)
    tree = fmm_mod.ATree(_t(xy), max_leaf, depth, BOX)
    uv = tree.velocity(_t(g), sigma, p, precision).cpu().numpy()
    ref = oracle_mod.afmm_velocity(xy, g, sigma, max_leaf, depth, p, BOX)
    assert rel_l2(uv, ref) < (1e-10 if precision == "fp64" else 1e-5)
    _check(tree, g, sigma, p, precision, dl, oracle_mod.afmm_grad(xy, g, sigma, max_leaf, depth, p, dl, BOX))
