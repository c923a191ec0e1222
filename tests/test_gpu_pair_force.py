"""The adjoint with respect to particles that move as evaluation point and source at once
(dl_dxy without its two parts), whose near field sums the pair force: the sum of the oracle's
two parts, at the leaf sizes where the mutual items and the target-centric units change, with
and without dL/dGamma, both trees; and with factors whose products leave FP32's range.

Tolerances: the repository's gates for the gradients (FP64 1e-9, mixed 1e-4).
"""
import numpy as np
import pytest

from conftest import rel_l2
from test_gpu_sparse_units import BOX, BWD, OPT_DENSE_LEAF, SIZES, _leaves, _t

pytestmark = pytest.mark.gpu


def _vjp(tree, g, sigma, p, precision, dl, with_gamma):
    import torch
    dg = torch.full((len(g),), np.nan, dtype=torch.float64, device="cuda") if with_gamma else None
    dx = torch.full((len(g), 2), np.nan, dtype=torch.float64, device="cuda")
    tree.transport_vjp(_t(g), sigma, p, precision, _t(dl), 1.0, 0, dg, dx)
    return (dg.cpu().numpy() if with_gamma else None), dx.cpu().numpy()


def _check(tree, g, sigma, p, precision, dl, refs, scale=1.0):
    for with_gamma in (False, True):
        dg, dx = _vjp(tree, g, sigma, p, precision, dl, with_gamma)
        assert rel_l2(dx / scale, refs[1] + refs[2]) < BWD[precision], (sigma, with_gamma)
        if with_gamma:
            assert rel_l2(dg, refs[0]) < BWD[precision], sigma


DENSE = [17, 64, 128, 65, 16, 15, 1, 200, 33, 32, 63, 0, 48, 80, 129, 31]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes,depth", [(SIZES, 3), (DENSE, 2), ([64] * 16, 2), ([0, 0, 5], 3), ([7, 0, 40], 1)],
                         ids=["ragged", "dense", "full", "corner", "no_far"])
def test_uniform(fmm_mod, oracle_mod, sizes, depth, precision):
    xy, g, r = _leaves(sizes, depth, 6)
    dl = r.standard_normal(xy.shape)
    for sigma in (0.3, 0.03, 0.004):  # the series everywhere; a few pairs; nearly all beyond the exponential
        tree = fmm_mod.Tree(_t(xy), depth, BOX)
        refs = oracle_mod.fmm_grad_full(xy, g, sigma, depth, 6, dl, BOX)
        for dense in (1, 32, 1 << 30):
            tree.set_option(OPT_DENSE_LEAF, dense)
            _check(tree, g, sigma, 6, precision, dl, refs)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("max_leaf", [3, 40, 130])
def test_adaptive(fmm_mod, oracle_mod, max_leaf, precision):
    r = np.random.Generator(np.random.PCG64(max_leaf))
    line = np.stack([0.5 + 0.002 * r.random(1500), 0.25 + 0.25 * r.random(1500)], axis=1)
    xy = np.concatenate([line, 0.1 + 0.3 * r.random((2000, 2)), r.random((60, 2))])
    g, dl = r.standard_normal(len(xy)), r.standard_normal(xy.shape)
    depth, p = 9, 8
    tree = fmm_mod.ATree(_t(xy), max_leaf, depth, BOX)
    for sigma in (0.02, 0.002, 0.0002):
        _check(tree, g, sigma, p, precision, dl, oracle_mod.afmm_grad(xy, g, sigma, max_leaf, depth, p, dl, BOX))


@pytest.mark.parametrize("kind", ["uniform", "adaptive"])
@pytest.mark.parametrize("sg,sq", [(1e-20, 1e-22), (1e15, 1e28), (1e-30, 1e25)])
def test_range_of_factors(fmm_mod, kind, sg, sq):
    """Mixed: products of Gamma and the cotangent outside FP32's range."""
    xy, g, r = _leaves(DENSE, 2, 7)
    dl = r.standard_normal(xy.shape)
    tree = fmm_mod.ATree(_t(xy), 40, 4, BOX) if kind == "adaptive" else fmm_mod.Tree(_t(xy), 2, BOX)
    want = _vjp(tree, g, 0.03, 6, "fp64", dl, True)
    dg, dx = _vjp(tree, sg * g, 0.03, 6, "mixed", sq * dl, True)
    assert rel_l2(dx / sg / sq, want[1]) < BWD["mixed"] and rel_l2(dg / sq, want[0]) < BWD["mixed"]


@pytest.mark.parametrize("kind", ["uniform", "adaptive"])
def test_replays(fmm_mod, kind):
    """Captured with dL/dGamma after a call without it: every replay has the eager bits."""
    import torch
    xy, g, r = _leaves(DENSE, 2, 8)
    dl = r.standard_normal(xy.shape)
    tree = fmm_mod.ATree(_t(xy), 40, 4, BOX) if kind == "adaptive" else fmm_mod.Tree(_t(xy), 2, BOX)
    _vjp(tree, g, 0.03, 6, "mixed", dl, False)
    gt, dt = _t(g), _t(dl)
    dg, dx = torch.empty_like(gt), torch.empty_like(dt)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tree.transport_vjp(gt, 0.03, 6, "mixed", dt, 1.0, 0, dg, dx)
    for k in range(3):
        d = dl * (1.0 + k)
        dt.copy_(_t(d))
        dg.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = dg.cpu().numpy(), dx.cpu().numpy()
        ref = _vjp(tree, g, 0.03, 6, "mixed", d, True)
        assert all(np.array_equal(a, b) for a, b in zip(got, ref)), k


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", ["uniform", "adaptive"])
def test_bits_of_every_schedule(fmm_mod, kind, precision):
    """The pair force beside the far chains, at every cap, and after them: one set of bits."""
    r = np.random.Generator(np.random.PCG64(12))
    xy, g, dl = r.random((6000, 2)), r.standard_normal(6000), r.standard_normal((6000, 2))
    tree = fmm_mod.ATree(_t(xy), 20, 6, BOX) if kind == "adaptive" else fmm_mod.Tree(_t(xy), 4, BOX)
    ref = _vjp(tree, g, 0.01, 9, precision, dl, True)
    for schedule in (0, 1) if kind == "uniform" else (None,):
        if schedule is not None:
            tree.set_option(1, schedule)
        for cap in (0, 1, 2, 3, 4, 5, 6):
            tree.set_option(8, cap)
            got = _vjp(tree, g, 0.01, 9, precision, dl, True)
            assert all(np.array_equal(a, b) for a, b in zip(got, ref)), (schedule, cap)
