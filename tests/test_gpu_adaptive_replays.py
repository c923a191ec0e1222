"""Adaptive tree, FP64: adjoint calls captured into a graph after an eager call of the position
derivative alone (the pair force), of its own route and of the separate parts: every replay has
the eager bits.
"""
import numpy as np
import pytest

from test_gpu_sparse_units import BOX, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("parts", [False, True], ids=["pair_force", "parts"])
def test_replays_after_pair_force(fmm_mod, parts):
    import torch
    r = np.random.Generator(np.random.PCG64(21))
    xy = np.concatenate([0.3 + 0.01 * r.standard_normal((1500, 2)), r.random((1500, 2))])
    g, dl = _t(r.standard_normal(3000)), r.standard_normal((3000, 2))
    dt = _t(dl)
    tree = fmm_mod.ATree(_t(xy), 40, 7, BOX)

    def call(d):
        if parts:
            return tree.velocity_backward(g, 0.002, 9, "fp64", d, need_src=True)
        dg, dx = torch.empty_like(g), torch.empty_like(d)
        tree.transport_vjp(g, 0.002, 9, "fp64", d, 1.0, 0, dg, dx)
        return dg, dx

    tree.transport_vjp(g, 0.002, 9, "fp64", dt, 1.0, 0, None, torch.empty_like(dt))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = call(dt)
    for k in range(3):
        dt.copy_(_t(dl * (1.0 + k)))
        graph.replay()
        torch.cuda.synchronize()
        got = [a.cpu().numpy() for a in captured]
        ref = [a.cpu().numpy() for a in call(_t(dl * (1.0 + k)))]
        assert all(np.array_equal(a, b) for a, b in zip(got, ref)), k
