"""Steps of the mutual near field's chunks of 16 sources: leaves around the chunk and tile sizes,
either tile of a pair in the lanes, every particle with its own circulation, forward against the
oracle.  A term added to another lane's sum shows in single particles, so the largest error counts.

Tolerances: the repository's gates for the near field (FP64 1e-12, mixed 1e-5), of the largest
velocity.
"""
import numpy as np
import pytest

from test_gpu_sparse_units import BOX, FWD, OPT_DENSE_LEAF, _leaves, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes", [[1, 15, 16, 17], [31, 32, 33, 47], [48, 49, 63, 64], [65, 2, 80, 113]])
def test_every_particle(fmm_mod, oracle_mod, sizes, precision):
    xy, g, _ = _leaves(sizes, 1, 11)
    tree = fmm_mod.Tree(_t(xy), 1, BOX)
    tree.set_option(OPT_DENSE_LEAF, 1)
    for sigma in (0.1, 0.01):  # every pair with the exponential; some tiles beyond it
        ref = oracle_mod.fmm_velocity(xy, g, sigma, 1, 6, BOX, parts=True)[0]
        near = tree.velocity_parts(_t(g), sigma, 6, precision)[0].cpu().numpy()
        assert np.abs(near - ref).max() < FWD[precision] * np.abs(ref).max(), sigma
