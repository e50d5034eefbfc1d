"""Rounding of the float64 symmetric sums.  Blocks of points carry forces (the adjoint: velocity gradients) of alternating
sign, so that the sums over a block are large and those over all points are not, and the order of the additions decides
the error.  Its size is taken from the same additions done in numpy, row by row: chunks of 64 columns (adjoint: 32) in
one chain each, the chunks of a block in another, and over the blocks exactly (the forward's fixed-point words) or in
three chains (the adjoint's three sets of atomic sums).  The kernel's columns, half of the pairs, have shorter chains,
so its rms error at a sample of points may be at most 1.5 times that; with the rows of a block in one chain it is
more than 4 times that."""
import math

import numpy as np
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

SAMPLE = 48


def _chain(x, start=None):
    return np.cumsum(x, axis=-1)[..., -1]  # float64, one addition after the other


def _problem(m, n, block):
    """m vesicles of n points on a lattice; s = +-1 by blocks."""
    k = np.arange(m * n)
    v, th = k // n, 2 * np.pi * (k % n) / n
    nx = int(math.ceil(math.sqrt(m)))
    X = np.stack([(v % nx) * 3.2 + 1.4 * np.cos(th), (v // nx) * 2.1 + 0.46 * np.sin(th)])
    s = np.where((k // block) % 2 == 0, 1.0, -1.0)
    return X, v, s


def _terms(X, v, s, i):
    """x-component of G(x_i - x_j) (s_j, 0) at every j of another vesicle, in long double."""
    r = X[:, i, None].astype(np.longdouble) - X.astype(np.longdouble)
    q = r[0] * r[0] + r[1] * r[1]
    other = v != v[i]
    q[~other] = 1
    return np.where(other, (-np.log(q) / 2 + r[0] * r[0] / q) * s, 0)


def _check(name, got, X, v, s, chunk, block, sets):
    P = X.shape[1]
    err, model = [], []
    for i in np.random.default_rng(3).choice(P, SAMPLE, replace=False):
        t = _terms(X, v, s, i)
        exact = t.sum()
        err.append(float(got[i] - exact))
        pad = np.zeros(-(-P // block) * block)
        pad[:P] = t.astype(np.float64)
        sums = _chain(_chain(pad.reshape(-1, block // chunk, chunk)))
        if sets:
            total = sum(_chain(sums[k::sets]) for k in range(sets))
        else:
            total = sums.astype(np.longdouble).sum()
        model.append(float(total - exact))
    rms = [math.sqrt(np.mean(np.square(x))) for x in (err, model)]
    say(f"{name}: rms error {rms[0]:.2e}, of the same additions {rms[1]:.2e}")
    assert rms[0] <= 1.5 * rms[1]


def test_forward():
    import torch
    import paper_2606_25569_amd as V
    X, v, s = _problem(1000, 100, 1024)  # blocks of 4 x 256 points, one unit per pair of blocks
    f = np.stack([s, np.zeros_like(s)])
    d = [torch.tensor(a, device="cuda") for a in (X, f, np.ones_like(s))]
    u = V.farfield_forward(d[0], d[0], d[1], d[2], np.arange(1001) * 100, 0.25 / math.pi, "fp64")
    _check("forward", u[0].cpu().numpy(), X, v, s, 64, 1024, 0)


def test_adjoint():
    import torch
    import paper_2606_25569_amd as V
    X, v, s = _problem(720, 100, 768)  # blocks of 3 x 256 points
    g = np.stack([s, np.zeros_like(s)])
    d = [torch.tensor(a, device="cuda") for a in (X, g, np.ones_like(s))]
    gf = V.farfield_backward_points(d[0], d[1], d[2], np.arange(721) * 100, 0.25 / math.pi, d[1], "fp64")[1]
    _check("adjoint", gf[0].cpu().numpy(), X, v, s, 32, 768, 3)
