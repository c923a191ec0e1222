"""Rows between user and sorted order on both sides of the sizes where they stop going directly
(2^20 rows forward, 2^19 adjoint): the same particles with and without one more far corner
particle give the same values to rounding, and a step equals base + h u.

Tolerance: 1e-12, a rounding of the sums per particle times the largest of their terms (FP64).
"""
import numpy as np
import pytest

from conftest import rel_l2
from test_gpu_sparse_units import BOX, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["uniform", "adaptive"])
@pytest.mark.parametrize("n", [1 << 19, 1 << 20])
def test_both_sides(fmm_mod, kind, n):
    import torch
    r = np.random.Generator(np.random.PCG64(n))
    xy = 0.01 + 0.98 * r.random((n + 1, 2))
    xy[n] = 0.999
    g, lam = r.standard_normal(n + 1) / n, r.standard_normal((n + 1, 2))
    g[n] = 0.0       # the extra particle moves nothing
    lam[n] = 0.0
    sigma, p, h = 0.002, 8, 0.25
    out = []
    for m in (n, n + 1):
        x, gt, lt = _t(xy[:m]), _t(g[:m]), _t(lam[:m])
        tree = fmm_mod.ATree(x, 64, 10, BOX) if kind == "adaptive" else fmm_mod.Tree(x, 7, BOX)
        u = tree.velocity(gt, sigma, p, "fp64")
        step = tree.transport_step(gt, sigma, p, "fp64", x, h)
        assert torch.equal(step, torch.addcmul(x, u, torch.full_like(u, h))) or \
            float((step - (x + h * u)).abs().max()) < 1e-15
        dg, dx = torch.empty_like(gt), torch.empty_like(x)
        tree.transport_vjp(gt, sigma, p, "fp64", lt, 1.0, 0, dg, dx)
        out.append([v[:n].cpu().numpy() for v in (u, dg, dx)])
        tree.close()
        del x, gt, lt, u, step, dg, dx
    for a, b in zip(*out):
        assert rel_l2(a, b) < 1e-12
