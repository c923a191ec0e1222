"""Mixed adjoint of moving particles with circulations near either end of FP32's range: dL/dGamma,
which sums the charges alone, is that of ordinary circulations, and dL/dx scales with them.

Tolerances: dL/dGamma a rounding of FP32 sums of 4000 terms (1e-5, powers of two change nothing);
dL/dx the repository's gate (1e-4).
"""
import numpy as np
import pytest

from conftest import rel_l2
from test_gpu_pair_force import _vjp
from test_gpu_sparse_units import BOX, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", [-122, -60, 60, 120])
@pytest.mark.parametrize("per_leaf", [4000, 20])
def test_circulations_at_the_ends_of_fp32(fmm_mod, per_leaf, exponent):
    depth = 1 if per_leaf == 4000 else 5
    r = np.random.Generator(np.random.PCG64(per_leaf))
    n = 4000 if depth == 1 else per_leaf << (2 * depth)
    xy = r.random((n, 2)) * (0.5 if depth == 1 else 1.0)
    g = 0.5 + 0.5 * r.random(n)
    dl = np.tile([0.3, 0.9], (n, 1))  # every pair of a particle at the rim adds up
    sigma = 0.2 if depth == 1 else 1.0 / 32
    tree = fmm_mod.Tree(_t(xy), depth, BOX)
    want = _vjp(tree, g, sigma, 8, "mixed", dl, True)
    dg, dx = _vjp(tree, np.ldexp(g, exponent), sigma, 8, "mixed", dl, True)
    assert rel_l2(dg, want[0]) < 1e-5
    # (equal cotangents: what is left of dL/dx is its roundoff beside these weights)
    dl2 = r.standard_normal((n, 2))
    want = _vjp(tree, g, sigma, 8, "mixed", dl2, True)
    dg, dx = _vjp(tree, np.ldexp(g, exponent), sigma, 8, "mixed", dl2, True)
    assert rel_l2(dg, want[0]) < 1e-5 and rel_l2(np.ldexp(dx, -exponent), want[1]) < 1e-4
