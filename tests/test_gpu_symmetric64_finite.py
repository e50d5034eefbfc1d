"""Float64 sums in the symmetric form with forces that are not finite or as large as float64 holds: the outputs that such
a force enters are not finite, those of its own vesicle keep their values, and large finite forces give finite sums, as
in the direct form (compared with it: 1e-12 of the largest value, as in test_gpu_symmetric64.py)."""
import numpy as np
import pytest

from tests.gpu_util import dev_inputs
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


def _inputs(bad):
    s = _ragged_suspension(seed=5, sizes=[64, 33, 0, 90, 47] * 20, spacing=3.5)  # 4,680 points
    X, f, w = dev_inputs(s)
    if bad == "large":
        f *= 1e303
    else:
        j = int(s.offsets[23]) + 40  # in the middle of a vesicle of 90 points
        f[1, j] = float(bad)
    return s, X, f, w


def _compare(got, ref):
    import torch
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(got), fin)
    assert fin.any()
    assert (got - ref)[fin].abs().max() <= 1e-12 * ref[fin].abs().max()


@pytest.mark.parametrize("bad", ["nan", "inf", "-inf", "large"])
def test_single(bad):
    import paper_2606_25569_amd as V
    s, X, f, w = _inputs(bad)
    ref = V.farfield_forward(X, X, f, w, s.offsets, 1.0, "fp64", config=dict(pair_form=1))
    _compare(V.farfield_forward(X, X, f, w, s.offsets, 1.0, "fp64"), ref)
    for T in (1, 2, 4):
        _compare(V.farfield_forward(X, X, f, w, s.offsets, 1.0, "fp64", config=dict(pair_form=2, targets_per_thread=T)),
                 ref)


@pytest.mark.parametrize("bad", ["nan", "inf", "large"])
def test_batched(bad):
    import paper_2606_25569_amd as V
    s, X, f, w = _inputs(bad)
    soff = np.array([0, 20, 21, 70, 100], np.int32)
    run = lambda cfg: V.BatchedProblem(X, X, f, w, s.offsets, soff, 1.0, "fp64", cfg).run().clone()  # noqa: E731
    _compare(run(None), run(dict(pair_form=1)))
