"""Mutual items of leaves of many tiles, cut into parts whose sums are added up afterwards: at the
tile counts where the ranges, the larger leaf of the two and the slots of a leaf with itself
change, forward and adjoint, against the oracle; the bits do not depend on the schedule.

Tolerances: the repository's gates for the near field (FP64 1e-12 of ragged leaves, mixed
1e-5) and for the gradients (FP64 1e-9, mixed 1e-4).
"""
import numpy as np
import pytest

from conftest import rel_l2
from test_gpu_pair_force import _check
from test_gpu_sparse_units import BOX, FWD, OPT_DENSE_LEAF, _leaves, _t

pytestmark = pytest.mark.gpu
OPT_SCHEDULE, OPT_NEAR_OCCUPANCY = 1, 8
SIZES = {"ragged": [700, 300, 257, 64, 256, 513, 31, 0, 255, 1, 320, 40, 200, 65, 448, 90],
         "corner": [0] * 15 + [1025], "row": [33, 1000, 0, 0], "equal": [256] * 4}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes", list(SIZES))
def test_against_oracle(fmm_mod, oracle_mod, sizes, precision):
    depth = 2 if len(SIZES[sizes]) > 4 else 1
    xy, g, r = _leaves(SIZES[sizes], depth, 9)
    dl = r.standard_normal(xy.shape)
    for sigma in (0.1, 0.01):  # every pair with the exponential; tiles beyond it
        tree = fmm_mod.Tree(_t(xy), depth, BOX)
        on = oracle_mod.fmm_velocity(xy, g, sigma, depth, 6, BOX, parts=True)[0]
        refs = oracle_mod.fmm_grad_full(xy, g, sigma, depth, 6, dl, BOX)
        for dense in (1, 32, 200):  # with and without target-centric units that are heavy themselves
            tree.set_option(OPT_DENSE_LEAF, dense)
            near = tree.velocity_parts(_t(g), sigma, 6, precision)[0].cpu().numpy()
            assert rel_l2(near, on) < FWD[precision], (sigma, dense)
            _check(tree, g, sigma, 6, precision, dl, refs)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_bits_of_every_launch(fmm_mod, precision):
    xy, g, r = _leaves(SIZES["ragged"], 2, 10)
    tree = fmm_mod.Tree(_t(xy), 2, BOX)
    ref = tree.velocity(_t(g), 0.03, 6, precision).cpu().numpy()
    for schedule in (0, 1):
        tree.set_option(OPT_SCHEDULE, schedule)
        for cap in (1, 3, 8):
            tree.set_option(OPT_NEAR_OCCUPANCY, cap)
            got = tree.velocity(_t(g), 0.03, 6, precision).cpu().numpy()
            assert np.array_equal(got, ref), (schedule, cap)
