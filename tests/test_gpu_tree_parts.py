"""The tree evaluations' parts of a leaf: leaves of every size from 1 to 70 points (one part up to 32, equal parts
above, from 8 to 16 lanes), few and many boxes per wavefront; rounding-level agreement with the oracles of the same tree
(1e-12 of max |u|, as in test_gpu_treecode.py)."""
import numpy as np
import pytest

from oracle import fmm as FM
from oracle import treecode as TC
from synth import suspension as S
from tests.gpu_util import dev_inputs, say

pytestmark = pytest.mark.gpu


def _clusters(first):
    """16 x 16 leaves at depth 4, 70 of them with 1 .. 70 points (small circles of up to 10 points around the leaf
    centres), the rest empty; two far points fix the root square."""
    rng = np.random.default_rng(first)
    sizes, centers = [1, 1], [[0.0, 0.0], [16.0, 16.0]]
    leaves = rng.permutation(255)[:70] + 1  # not the corner leaf of the first point
    for k, leaf in enumerate(leaves[leaves != 255]):
        left = first + k
        while left > 0:
            sizes.append(min(10, left))
            left -= sizes[-1]
            centers.append([leaf // 16 + rng.uniform(0.25, 0.75), leaf % 16 + rng.uniform(0.25, 0.75)])
    m = len(sizes)
    return S._assemble(rng, np.array(centers), np.tile([0.2, 0.12], (m, 1)) * (np.array(sizes) > 1)[:, None] + 1e-9,
                       rng.uniform(0, 6.28, m), np.array(sizes), "k4", 0.2, 1.0, 16.0)


@pytest.mark.parametrize("order", [5, 20, 31, 32, 48])
def test_leaf_sizes(order):
    import torch
    import paper_2606_25569_amd as V
    s = _clusters(1)
    X, f, w = dev_inputs(s)
    for label, run, oracle in (("treecode", V.farfield_treecode, TC.treecode), ("fmm", V.farfield_fmm, FM.fmm)):
        got = run(X, f, w, s.offsets, s.mu, order, 4)
        assert torch.equal(got, run(X, f, w, s.offsets, s.mu, order, 4))
        ref = oracle(s.X, s.f, s.w, s.offsets, s.mu, order, 4)
        err = np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max()
        say(f"{label} order={order} P={s.n_points}: {err:.2e}")
        assert err <= 1e-12
