"""The first call after a rebuild, captured: it clears what the old tree left in the multipoles of
cells that are now empty, at every replay (the eager bits, also with another tree that shares the
workspace in between).
"""
import numpy as np
import pytest

from test_gpu_sparse_units import BOX, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_capture_after_rebuild(fmm_mod, precision):
    import torch
    r = np.random.Generator(np.random.PCG64(51))
    n, depth, p, sigma = 6000, 6, 9, 0.004
    everywhere, corner = _t(r.random((n, 2))), _t(0.05 + 0.3 * r.random((n, 2)))
    g, out = _t(r.standard_normal(n)), torch.empty(n, 2, dtype=torch.float64, device="cuda")
    fresh, other = fmm_mod.Tree(corner, depth, BOX), fmm_mod.Tree(everywhere, depth, BOX)
    tree = fmm_mod.Tree(everywhere, depth, BOX)
    other.share_workspace(tree)
    tree.velocity(g, sigma, p, precision)
    tree.rebuild(corner, BOX)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tree.velocity(g, sigma, p, precision, out=out)
    for k in range(4):
        g.copy_(_t(r.standard_normal(n)))
        if k % 2:
            other.velocity(g, sigma, p, precision)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, fresh.velocity(g, sigma, p, precision)), k
