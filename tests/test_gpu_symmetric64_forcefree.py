"""Rounding of the float64 symmetric sums over vesicles without net force: the partial sums over a vesicle are tens of
times its terms and return to almost nothing, so that the error counts the roundings at their size.  Its size is taken
from the same additions in numpy, row by row: the terms of the matrix's diagonal and the others in a chain each over a
chunk of 64 columns (adjoint: 32), the chunks' sums in one over a block, the blocks' exactly (adjoint: in three chains).
The kernel's columns, half of the pairs, have chains of 20 additions at most: with half of the rows' variance for them the
rms error is sqrt(3 / 4) of that, and may be 0.9 of it at a sample of points (the adjoint's all of it, as the order of its
atomic additions differs from run to run).  Both terms of every pair added to one sum exceed it."""
import math

import numpy as np
import pytest

from tests.gpu_util import say
from tests.test_gpu_symmetric64_rounding import _chain, _problem

pytestmark = pytest.mark.gpu

SAMPLE = 48


def _check(name, got, X, v, f, chunk, block, sets):
    P = X.shape[1]
    err, model = [], []
    fl = f.astype(np.longdouble)
    for i in np.random.default_rng(3).choice(P, SAMPLE, replace=False):
        other = v != v[i]
        rl = X[:, i, None].astype(np.longdouble) - X.astype(np.longdouble)
        ql = rl[0] * rl[0] + rl[1] * rl[1]
        ql[~other] = 1
        exact = np.where(other, (-np.log(ql) / 2 + rl[0] * rl[0] / ql) * fl[0] + rl[0] * rl[1] / ql * fl[1], 0).sum()
        err.append(float(got[i] - exact))
        r = X[:, i, None] - X
        q = r[0] * r[0] + r[1] * r[1]
        q[~other] = 1
        sums = 0.0
        for term in ((-0.5 * np.log(q) + r[0] * r[0] / q) * f[0], r[0] * r[1] / q * f[1]):
            padded = np.zeros(-(-P // block) * block)
            padded[:P] = np.where(other, term, 0)
            sums = sums + _chain(padded.reshape(-1, block // chunk, chunk))
        sums = _chain(sums)
        total = sum(_chain(sums[k::sets]) for k in range(sets)) if sets else sums.astype(np.longdouble).sum()
        model.append(float(total - exact))
    rms = [math.sqrt(np.mean(np.square(x))) for x in (err, model)]
    say(f"{name}: rms error {rms[0]:.2e}, of the same additions {rms[1]:.2e}")
    assert rms[0] <= (1.0 if sets else 0.9) * rms[1]


def _force_free(m, n, block):
    X, v, _ = _problem(m, n, block)
    th = 2 * np.pi * (np.arange(m * n) % n) / n
    rng = np.random.default_rng(1)
    a = rng.standard_normal((2, 4, m))[:, :, v]
    f = a[:, 0] * np.cos(th) + a[:, 1] * np.sin(th) + a[:, 2] * np.cos(2 * th) + a[:, 3] * np.sin(2 * th)
    return X, v, np.ascontiguousarray(f)


def test_forward():
    import torch
    import paper_2606_25569_amd as V
    X, v, f = _force_free(1000, 100, 1024)  # blocks of 4 x 256 points
    d = [torch.tensor(a, device="cuda") for a in (X, f, np.ones(X.shape[1]))]
    u = V.farfield_forward(d[0], d[0], d[1], d[2], np.arange(1001) * 100, 0.25 / math.pi, "fp64")
    _check("forward", u[0].cpu().numpy(), X, v, f, 64, 1024, 0)


def test_adjoint():
    import torch
    import paper_2606_25569_amd as V
    X, v, g = _force_free(720, 100, 768)  # blocks of 3 x 256 points
    d = [torch.tensor(a, device="cuda") for a in (X, g, np.ones(X.shape[1]))]
    gf = V.farfield_backward_points(d[0], d[1], d[2], np.arange(721) * 100, 0.25 / math.pi, d[1], "fp64")[1]
    _check("adjoint", gf[0].cpu().numpy(), X, v, g, 32, 768, 3)
