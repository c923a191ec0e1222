"""The cells of the adaptive device build, which every particle finds from its key and the key
max_leaf places on, at the edges of that rule: as many particles as a leaf may hold and one more,
coincident particles, runs that end within max_leaf places of the array's ends, a chain of
single-child cells, the deepest level full.  The structure and the velocities are those of the
host build, bit for bit.
"""
import numpy as np
import pytest

from test_gpu_adaptive import _same_atree, _t

pytestmark = pytest.mark.gpu


def _points(kind, n):
    r = np.random.Generator(np.random.PCG64(n))
    if kind == "same":  # the square is the unit square's: two corners besides
        return np.concatenate([np.full((n - 2, 2), 0.3), [[0.0, 0.0], [1.0, 1.0]]])
    if kind == "corner":
        return np.concatenate([1e-4 * r.random((n - 1, 2)), [[1.0, 1.0]]])
    if kind == "line":
        return np.stack([np.linspace(0.0, 1.0, n), np.full(n, 0.5)], axis=1)
    return r.random((n, 2))


@pytest.mark.parametrize("kind,n,max_leaf,depth", [
    ("random", 1, 4, 5), ("random", 4, 4, 5), ("random", 5, 4, 5), ("random", 9, 8, 15), ("random", 700, 1, 15),
    ("random", 700, 699, 4), ("random", 2049, 1, 4), ("same", 40, 4, 15), ("same", 6, 3, 2), ("corner", 300, 7, 15),
    ("corner", 66, 64, 12), ("line", 1000, 2, 10), ("line", 257, 16, 8)])
def test_cells(fmm_mod, kind, n, max_leaf, depth):
    x = _t(_points(kind, n))
    g = _t(np.random.Generator(np.random.PCG64(n + 1)).standard_normal(n))
    td = fmm_mod.ATree(x, max_leaf, depth, (0.0, 0.0, 1.0), builder="device")
    th = fmm_mod.ATree(x, max_leaf, depth, (0.0, 0.0, 1.0), builder="host")
    _same_atree(td, th, g, 0.01, 8)
