"""fmm_velocity_noalloc at the end of its range: mixed calls that fit the static workspace only
with levels up to L_c in FP64 are taken (for every L_c), and agree with the FP64 velocities.

Tolerance: the repository's gate for mixed velocities (1e-5).
"""
import numpy as np
import pytest

from conftest import rel_l2
from test_gpu_sparse_units import BOX, _t
from test_zz_no_alloc import _call

pytestmark = pytest.mark.gpu
LIMIT, OPT_COARSE_LEVEL, OPT_SCHEDULE = 128 << 20, 2, 1


def _cells(level):
    """Cells above `level`, all levels."""
    return (4 ** level - 1) // 3


def _bytes(n, depth, p, split):
    """The workspace of a mixed call over a tree with mutual items and its coordinates made."""
    def pad(b):
        return (b + 255) // 256 * 256
    d = _cells(split + 1) * p + 64
    f = (_cells(depth + 1) - _cells(split + 1)) * p + 64
    return pad(4 * n) + 2 * pad(16 * n) + pad(72 * n) + 2 * pad(16 * d) + 2 * pad(8 * f)


@pytest.mark.parametrize("lc", [1, 2, 3])
def test_levels_at_the_limit(fmm_mod, lc):
    import torch
    from paper_1008_2410_amd import _lib
    lib = _lib.load()
    depth, p, sigma = 7, 16, 0.001
    n = (LIMIT - _bytes(0, depth, p, 5)) // 108 + 1000  # 108 bytes a particle, 20 KiB a term for levels 4 and 5
    assert _bytes(n, depth, p, 5) > LIMIT >= _bytes(n, depth, p, lc)
    r = np.random.Generator(np.random.PCG64(74))
    xy, g = _t(r.random((n, 2))), _t(r.standard_normal(n) / n)
    tree = fmm_mod.Tree(xy, depth, BOX)
    assert tree.near_plan()["mutual_items"] > 0
    ref = tree.velocity(g, sigma, p, "fp64").cpu().numpy()
    tree.velocity(g, sigma, p, "mixed")  # the tables and the coordinates
    tree.set_option(OPT_COARSE_LEVEL, lc)
    for schedule in (0, 1):
        tree.set_option(OPT_SCHEDULE, schedule)
        out = torch.full((n, 2), float("nan"), dtype=torch.float64, device="cuda")
        rc, _ = _call(lib, "fmm_velocity_noalloc", tree, g, sigma, p, _lib.FMM_MIXED, out)
        assert rc == _lib.FMM_OK, lib.fmm_last_error()
        assert rel_l2(out.cpu().numpy(), ref) < 1e-5, schedule
    tree.close()
