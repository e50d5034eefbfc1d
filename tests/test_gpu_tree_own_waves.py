"""The trees' own-vesicle terms, 64 targets and 64 points at a time by two wavefronts per vesicle: vesicles at the edges
of those counts, odd and even numbers of vesicles; rounding-level agreement with the oracles of the same tree (1e-12 of
max |u|, as in test_gpu_treecode.py)."""
import numpy as np
import pytest

from oracle import fmm as FM
from oracle import treecode as TC
from synth import suspension as S
from tests.gpu_util import dev_inputs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[63, 64, 65], [1, 129, 0, 191], [128, 192, 193, 0, 2]])
@pytest.mark.parametrize("depth", [2, 4])
def test_edges(sizes, depth):
    import paper_2606_25569_amd as V
    rng = np.random.default_rng(sum(sizes))
    m = len(sizes)
    centers = np.array([[14.0 * (k % 2), 11.0 * (k // 2)] for k in range(m)])
    axes = np.tile([5.0, 3.5], (m, 1))
    s = S._assemble(rng, centers, axes, rng.uniform(0, 6.28, m), np.array(sizes), "k4", 0.2, 1.0, 40.0)
    X, f, w = dev_inputs(s)
    for label, run, oracle in (("treecode", V.farfield_treecode, TC.treecode), ("fmm", V.farfield_fmm, FM.fmm)):
        got = run(X, f, w, s.offsets, s.mu, 16, depth).cpu().numpy()
        ref = oracle(s.X, s.f, s.w, s.offsets, s.mu, 16, depth)
        err = np.abs(got - ref).max() / np.abs(ref).max()
        say(f"{label} {sizes} depth={depth}: {err:.2e}")
        assert err <= 1e-12
