"""Trees far from unit scale, at orders whose padded rows (multiples of 8 above the order) or powers of box widths leave
the float64 range before the moments do.  Scaling the coordinates by a power of two scales every box, moment and
coefficient exactly, so that u(s X) = u(X) - ln s / (4 pi mu) sum_{j of other vesicles} F_j up to the rounding of the
logarithms: at most 1,000 sequential additions per value (9 leaves, 27 boxes a level, the series) of terms of at most
(|ln s| + 8) |F_j|, half an ulp each."""
import math

import numpy as np
import pytest

from tests.gpu_util import dev_inputs, say
from tests.test_gpu_tree_chunks import _susp

pytestmark = pytest.mark.gpu

DEPTH = 4


def _check(name, run, order, side):
    import torch
    s = _susp(700)
    X, f, w = dev_inputs(s)
    extent = float(np.ptp(s.X, axis=1).max())
    e = round(math.log2(side / extent))
    X *= side * 2.0**-e / extent  # the root square of the scaled points has this side
    u = run(X, f, w, s.offsets, s.mu, order, DEPTH).cpu().numpy()
    v = run(torch.ldexp(X, torch.tensor(e, device=X.device)), f, w, s.offsets, s.mu, order, DEPTH).cpu().numpy()
    F = s.w * s.f
    own = np.add.reduceat(F, s.offsets[:-1], axis=1)
    other = F.sum(axis=1, keepdims=True) - np.repeat(own, s.sizes(), axis=1)
    lns = e * math.log(2.0)
    want = u - lns * other / (4 * math.pi * s.mu)
    tol = 1000 * 2.0**-53 * (abs(lns) + 8) * np.abs(F).sum() / (4 * math.pi * s.mu)
    err = np.abs(v - want).max()
    say(f"{name} order={order} side={side:.2e}: {err:.2e} of {tol:.2e}, max |u| {np.abs(want).max():.2e}")
    assert err <= tol


@pytest.mark.parametrize("order,side", [(32, 6.5e8), (40, 3e7), (48, 4e6), (48, 7.2e-6), (30, 1e9), (30, 1e-8)])
def test_fmm(order, side):
    import paper_2606_25569_amd as V
    _check("fmm", V.farfield_fmm, order, side)


@pytest.mark.parametrize("order,side", [(32, 6.5e8), (48, 4e6), (40, 1e-12), (48, 1e-11)])
def test_treecode(order, side):
    import paper_2606_25569_amd as V
    _check("treecode", V.farfield_treecode, order, side)
