"""The float64 logarithm of the direct sums, of their adjoint and of the fast multipole method's direct part: -ln d of
4,096 distances with d^2 in [2^9, 2^10), one pair each, without bias.  One target's value carries up to half an ulp of
its size (2.2e-16) and the table's error (about 1e-16), whose mean over the distances is below 1e-17; ln 2 rounded to
one word moves every value by 10 x 1.2e-17."""
import math

import numpy as np
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

N = 4096


def _direct(V, X, f, w, off, mu):
    return V.farfield_forward(X, X, f, w, off, mu, "fp64", config=dict(pair_form=1, block_threads=256))[0, :N]


def _small(V, X, f, w, off, mu):
    return V.farfield_forward(X[:, 1:].contiguous(), X[:, 1:].contiguous(), f[:, 1:].contiguous(), w[1:],
                              np.array([0, N - 1, N]), mu, "fp64")[0, :N - 1]


def _adjoint(V, X, f, w, off, mu):
    return V.farfield_backward(X, X, f, w, off, mu, f, "fp64", (False, False, True, False))[2][0, :N]


def _fmm(V, X, f, w, off, mu):
    return V.farfield_fmm(X, f, w, off, mu, 8, 0)[0, :N]


@pytest.mark.parametrize("run", [_direct, _small, _adjoint, _fmm])
def test_bias(run):
    import torch
    import paper_2606_25569_amd as V
    # targets (0, d), the source (0, 0) with force (1, 0): u_x = -ln d, and d^2 is exact
    d = np.round(np.linspace(2.0**4.5 + 1e-3, 2.0**5 - 1e-3, N) * 2**20) / 2**20
    X = np.zeros((2, N + 1))
    X[1, :N] = d
    f = np.zeros_like(X)
    f[0, N] = 1.0
    t = [torch.tensor(a, device="cuda") for a in (X, f, np.ones(N + 1))]
    u = run(V, *t, np.array([0, N, N + 1]), 0.25 / math.pi).cpu().numpy()
    err = (u.astype(np.longdouble) + np.log(d[N - u.size:].astype(np.longdouble))).astype(np.float64)
    say(f"{run.__name__}: mean {err.mean():.1e}, rms {np.sqrt(np.mean(err * err)):.1e}, max {np.abs(err).max():.1e}")
    assert np.abs(err).max() <= 3.5e-16
    assert abs(err.mean()) <= 4e-17
