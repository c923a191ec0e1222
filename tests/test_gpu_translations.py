"""Far field against the oracle at the edges of the translation kernels: expansion orders on
both sides of each table size (8, 12, 16, 24 and 32 terms), trees of 2 to 8 levels (levels
in one launch, level by level and wide levels with the L2L taken along), ragged leaves and
empty cells, both trees.

Tolerance: an FP64 local is a chain of at most 7 levels of 27 products of 2p terms, at most
27 x 64 x 7 = 12096 additions of relative rounding 1.1e-16: 1.4e-12 of the largest partial
sums, a factor 10 for their cancellation.  The mixed form keeps its gate of 1e-5.
"""
import numpy as np
import pytest

from conftest import rel_l2

pytestmark = pytest.mark.gpu
BOX = (0.0, 0.0, 1.0)
TOL = {"fp64": 1.4e-11, "mixed": 1e-5}


def _t(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def _cloud(n, seed, clustered):
    r = np.random.Generator(np.random.PCG64(seed))
    xy = r.random((n, 2))
    if clustered:  # a quarter of the square dense, the rest mostly empty cells
        xy[: 7 * n // 8] *= 0.25
    return xy, r.standard_normal(n) / n


@pytest.mark.parametrize("precision,depth,n,p,clustered", [
    ("fp64", 2, 37, 1, False), ("fp64", 2, 300, 8, False), ("fp64", 2, 300, 17, False), ("fp64", 3, 500, 9, True),
    ("fp64", 4, 2000, 13, False), ("fp64", 5, 3000, 24, True), ("fp64", 6, 9000, 16, True), ("fp64", 6, 9000, 25, False),
    ("fp64", 7, 40000, 12, False), ("fp64", 7, 40000, 32, True), ("fp64", 8, 150000, 10, False),
    ("mixed", 5, 3000, 7, False), ("mixed", 6, 9000, 12, True), ("mixed", 7, 40000, 16, False),
    ("mixed", 7, 40000, 20, True), ("mixed", 8, 400000, 13, False)])
def test_uniform_far_field(fmm_mod, oracle_mod, precision, depth, n, p, clustered):
    xy, g = _cloud(n, 31 * depth + p, clustered)
    sigma = 0.05 / 2 ** depth
    tree = fmm_mod.Tree(_t(xy), depth, BOX)
    far = tree.velocity_parts(_t(g), sigma, p, precision)[1].cpu().numpy()
    ref = oracle_mod.fmm_velocity(xy, g, sigma, depth, p, BOX, parts=True)[1]
    err = rel_l2(far, ref)
    print(f"{precision} depth {depth} p {p}: far rel-L2 {err:.2e}", flush=True)
    assert err < TOL[precision]


@pytest.mark.parametrize("n,max_leaf,depth,p", [(400, 8, 3, 8), (3000, 4, 9, 9), (9000, 16, 8, 13), (9000, 16, 8, 17),
                                                (30000, 8, 10, 25), (200000, 16, 10, 16)])
def test_adaptive_far_field(fmm_mod, oracle_mod, n, max_leaf, depth, p):
    r = np.random.Generator(np.random.PCG64(n + p))
    xy = np.concatenate([r.random((n // 2, 2)), 0.3 + 0.004 * r.standard_normal((n - n // 2, 2))])
    g = r.standard_normal(n) / n
    sigma = 0.05 / 2 ** depth
    tree = fmm_mod.ATree(_t(xy), max_leaf, depth, BOX)
    uv = tree.velocity(_t(g), sigma, p, "fp64").cpu().numpy()
    ref = oracle_mod.afmm_velocity(xy, g, sigma, max_leaf, depth, p, BOX)
    err = rel_l2(uv, ref)
    print(f"adaptive depth {depth} p {p}: rel-L2 {err:.2e}", flush=True)
    assert err < TOL["fp64"]
