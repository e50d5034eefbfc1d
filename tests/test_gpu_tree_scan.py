"""Deep trees, whose leaf counts are scanned in one pass of 4,096 leaves (depth 6) and in four (depth 7): both tree
methods against the direct float64 oracle.  The expansions converge by a factor of at least 0.55 per order at the
worst separation of the interaction lists, 0.55^31 < 1e-8 at order 30; the bar is 1e-6 of max |u|."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import suspension as S
from tests.gpu_util import dev_inputs, rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth", [6, 7])
def test_deep_tree(depth):
    import paper_2606_25569_amd as V
    s = S.rsa_suspension(31, 60, 40, 0.3)
    X, f, w = dev_inputs(s)
    ref = O.farfield_suspension(s.X, s.f, s.w, s.offsets, s.mu)
    for run in (V.farfield_treecode, V.farfield_fmm):
        err, _ = rel_err(run(X, f, w, s.offsets, s.mu, 30, depth).cpu().numpy(), ref)
        say(f"{run.__name__} depth={depth}: {err:.2e}")
        assert err <= 1e-6
