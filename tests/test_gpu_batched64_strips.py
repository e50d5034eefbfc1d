"""Batched float64 sums at every number of column strips that the launch rule chooses (16, 8, 4, 2, 1 and, for large
suspensions, two targets per thread), with suspensions below and above the rule's mean and empty ones among them, and
plans with eight lanes and with a wavefront per suspension; against the direct form (1e-12 of the largest value, as in
test_gpu_batched.py)."""
import numpy as np
import pytest

from tests.gpu_util import dev_inputs
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,m,n", [(3, 2, 16), (3, 40, 8), (64, 2, 17), (96, 4, 32), (100, 10, 20), (300, 3, 43),
                                   (130, 9, 32), (260, 9, 32), (1030, 2, 16), (5, 30, 64)])
def test_against_direct(S, m, n):
    import torch
    import paper_2606_25569_amd as V
    rng = np.random.default_rng(S)
    per = rng.integers(max(0, m // 2), m + m // 2 + 1, S)
    per[S // 2] = 0
    sizes = rng.integers(max(1, n - 3), n + 4, int(per.sum())).tolist()
    s = _ragged_suspension(seed=S, sizes=sizes, spacing=3.5)
    X, f, w = dev_inputs(s)
    soff = np.concatenate([[0], np.cumsum(per)]).astype(np.int32)
    mu = rng.uniform(0.5, 2.0, S)
    b = V.BatchedProblem(X, X, f, w, s.offsets, soff, mu, "fp64")
    u = b.run().clone()
    assert torch.equal(u, b.run())
    ref = V.BatchedProblem(X, X, f, w, s.offsets, soff, mu, "fp64", dict(pair_form=1)).run()
    assert (u - ref).abs().max() <= 1e-12 * ref.abs().max()
