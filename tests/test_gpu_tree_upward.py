"""The trees' moments: every number of orders per lane and of matrix tiles (orders on both sides of multiples of 8 and
16), depths whose coarser levels take one or two launches, empty boxes, and coordinates far from 1; rounding-level
agreement with the oracles of the same tree (1e-12 of max |u|, as in test_gpu_treecode.py)."""
import numpy as np
import pytest

from oracle import fmm as FM
from oracle import treecode as TC
from tests.gpu_util import dev_inputs, say
from tests.test_gpu_tree_chunks import _susp

pytestmark = pytest.mark.gpu


def _check(s, order, depth, name, fmm=True):
    import torch
    import paper_2606_25569_amd as V
    X, f, w = dev_inputs(s)
    both = (("treecode", V.farfield_treecode, TC.treecode), ("fmm", V.farfield_fmm, FM.fmm))
    for label, run, oracle in both if fmm else both[:1]:
        got = run(X, f, w, s.offsets, s.mu, order, depth)
        assert torch.equal(got, run(X, f, w, s.offsets, s.mu, order, depth))
        ref = oracle(s.X, s.f, s.w, s.offsets, s.mu, order, depth)
        err = np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max()
        say(f"{label} {name} depth={depth} order={order}: {err:.2e}")
        assert err <= 1e-12


@pytest.mark.parametrize("order", [1, 6, 7, 8, 15, 16, 17, 23, 24, 31, 32, 39, 40, 47, 48])
def test_orders(order):
    _check(_susp(700), order, 4, "orders")


@pytest.mark.parametrize("depth", [2, 3, 5, 6])
def test_depths(depth):
    _check(_susp(1500), 13, depth, "depths")


@pytest.mark.parametrize("scale", [1e-5, 1e5])
def test_scaled(scale):
    """On the treecode, whose oracle keeps its accuracy at these scales (at 1e5 the fast multipole oracle's own error
    against the exact sum, 1.8e-12, is twice the GPU's)."""
    s = _susp(700)
    s.X = s.X * scale
    s.w = s.w * scale
    _check(s, 30, 4, f"scaled {scale:g}", fmm=False)
