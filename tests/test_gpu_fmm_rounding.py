"""Rounding of the fast multipole evaluation: one distant vesicle carries a force a million times the others', so that a
target's far part is huge and its direct part, over a thousand terms for each of a lane's sums, is not.  Added to the
far part one by one those terms would round over a thousand times at its size (an rms error of sqrt(1125 / 12) = 9.7
units in the last place); summed by themselves, fewer than 40 additions see it (levels, polynomial, groups, scale):
sqrt(40 / 12) = 1.8, with a margin 3."""
import math

import numpy as np
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def test_far_part_last():
    import torch
    import paper_2606_25569_amd as V
    rng = np.random.default_rng(7)
    n, per = 16000, 16
    c = rng.uniform(0.3, 15.7, (2, n // per))
    X = np.repeat(c, per, axis=1) + rng.uniform(-0.1, 0.1, (2, n))
    big = np.array([[2.0, 2.01, 2.0], [2.0, 2.0, 2.01]])     # about the centre of the lowest leaf of a 4 x 4 tree
    corners = np.array([[0.0, 16.0], [0.0, 16.0]])           # two vesicles of one point each
    X = np.concatenate([X, big, corners], axis=1)
    off = np.concatenate([np.arange(0, n + 1, per), [n + 3, n + 4, n + 5]]).astype(np.int32)
    f = rng.choice([-1.0, 1.0], X.shape)
    f[:, n:] = 0.0
    f[:, n:n + 3] = [[1e6], [-1e6]]
    vid = np.repeat(np.arange(off.size - 1), np.diff(off))
    t = [torch.tensor(a, device="cuda") for a in (X, f, np.ones(X.shape[1]))]
    u = V.farfield_fmm(*t, off, 0.25 / math.pi, 48, 2).cpu().numpy()
    # the leaf opposite: the expansions' truncation is below (0.2)^48 there
    idx = np.flatnonzero((X[0, :n] > 12) & (X[1, :n] > 12))[:64]
    err = []
    for i in idx:
        r = X[:, i, None].astype(np.longdouble) - X.astype(np.longdouble)
        q = r[0] * r[0] + r[1] * r[1]
        other = vid != vid[i]
        q[~other] = 1
        b = (r[0] * f[0] + r[1] * f[1]) / q
        ref = [np.where(other, -np.log(q) / 2 * f[k] + b * r[k], 0).sum() for k in (0, 1)]
        err.append([float((u[k, i] - ref[k]) / np.spacing(abs(float(ref[k])))) for k in (0, 1)])
    rms = math.sqrt(np.mean(np.square(err)))
    say(f"fmm: rms error {rms:.2f} units in the last place of {np.abs(u[:, idx]).max():.1e}")
    assert rms <= 3.0
