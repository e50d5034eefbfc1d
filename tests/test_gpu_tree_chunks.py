"""The tree evaluations at the edges of their wavefront chunks: point counts on both sides of the treecode's choice of
lanes per group, and leaves of a few points up to several chunks; rounding-level agreement with the oracles of the
same tree (1e-12 of max |u|, as in test_gpu_treecode.py)."""
import numpy as np
import pytest

from oracle import fmm as FM
from oracle import treecode as TC
from tests.gpu_util import dev_inputs, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


def _susp(total):
    rng = np.random.default_rng(total)
    sizes = []
    while sum(sizes) < total:
        sizes.append(min(int(rng.integers(1, 40)), total - sum(sizes)))
    return _ragged_suspension(seed=total, sizes=sizes, spacing=3.5)


# 44 points per leaf is the treecode's line: 704 / 705 at depth 2, 176 / 177 at depth 1
@pytest.mark.parametrize("total,depth", [(15, 1), (60, 2), (176, 1), (177, 1), (513, 2), (704, 2), (705, 2), (1300, 2),
                                         (900, 3), (2817, 3)])
@pytest.mark.parametrize("order", [1, 11, 32])
def test_chunk_edges(total, depth, order):
    import torch
    import paper_2606_25569_amd as V
    s = _susp(total)
    X, f, w = dev_inputs(s)
    got = V.farfield_treecode(X, f, w, s.offsets, s.mu, order, depth)
    again = V.farfield_treecode(X, f, w, s.offsets, s.mu, order, depth)
    assert torch.equal(got, again)
    ref = TC.treecode(s.X, s.f, s.w, s.offsets, s.mu, order, depth)
    err = np.abs(got.cpu().numpy() - ref).max()
    say(f"treecode P={total} depth={depth} order={order}: {err:.2e}")
    assert err <= 1e-12 * np.abs(ref).max()  # zero for a single vesicle
    got = V.farfield_fmm(X, f, w, s.offsets, s.mu, order, depth).cpu().numpy()
    ref = FM.fmm(s.X, s.f, s.w, s.offsets, s.mu, order, depth)
    err = np.abs(got - ref).max()
    say(f"fmm P={total} depth={depth} order={order}: {err:.2e}")
    assert err <= 1e-12 * np.abs(ref).max()
