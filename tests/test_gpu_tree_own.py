"""The trees' own-vesicle correction: vesicles much larger than a leaf and than a chunk of points, in curve order (long
runs of one leaf) and in random order (every point a run of its own, many far stretches); rounding-level agreement
with the oracles of the same tree (1e-12 of max |u|, as in test_gpu_treecode.py)."""
import numpy as np
import pytest

from oracle import fmm as FM
from oracle import treecode as TC
from synth import suspension as S
from tests.gpu_util import dev_inputs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order_of_points", ["curve", "random"])
@pytest.mark.parametrize("depth", [2, 3, 5])
def test_large_vesicles(order_of_points, depth):
    import paper_2606_25569_amd as V
    rng = np.random.default_rng(8)
    sizes = np.array([700, 7, 128, 129, 1, 257])
    centers = np.array([[0.0, 0.0], [15.0, 0.0], [0.0, 12.0], [15.0, 12.0], [8.0, 6.0], [24.0, 6.0]])
    axes = np.array([[6.0, 4.0], [1.2, 0.5], [5.0, 3.0], [5.0, 3.0], [0.5, 0.5], [3.0, 5.0]])
    s = S._assemble(rng, centers, axes, rng.uniform(0, 6.28, 6), sizes, "k4", 0.2, 1.0, 40.0)
    if order_of_points == "random":
        perm = np.concatenate([a + rng.permutation(b - a) for a, b in zip(s.offsets[:-1], s.offsets[1:])])
        s.X, s.f, s.w = s.X[:, perm].copy(), s.f[:, perm].copy(), s.w[perm].copy()
    X, f, w = dev_inputs(s)
    for label, run, oracle in (("treecode", V.farfield_treecode, TC.treecode), ("fmm", V.farfield_fmm, FM.fmm)):
        got = run(X, f, w, s.offsets, s.mu, 16, depth).cpu().numpy()
        ref = oracle(s.X, s.f, s.w, s.offsets, s.mu, 16, depth)
        err = np.abs(got - ref).max() / np.abs(ref).max()
        say(f"{label} {order_of_points} depth={depth}: {err:.2e}")
        assert err <= 1e-12
