"""Membrane force and near layers on the routes that the sizes choose: many small vesicles (the vector form, with larger
ones beside them), many of 129 to 256 points (two wavefronts each, with smaller and larger ones beside them), neighbours
and every second vesicle above 128 points, and every number of points up to 17.  Bars are those of test_gpu_spectral.py
and test_gpu_rbf.py."""
import numpy as np
import pytest

from oracle import nearfield_rbf as NR
from tests.gpu_util import say
from tests.test_gpu_rbf import _curves as weighted_curves
from tests.test_gpu_rbf import _layer_tol
from tests.test_gpu_spectral import EPS, _centred_reference, _curves

pytestmark = pytest.mark.gpu

CASES = {
    "small": [3, 5, 8, 24, 12, 17, 1, 0, 2, 16] * 210,
    "small and large": [8] * 1500 + [63, 64, 65, 128, 129, 300] + [7] * 1000,
    "two wavefronts": [129, 200, 256, 130, 255] * 206 + [100, 257, 40, 300, 0, 3],
    "neighbours": [32] * 300 + [150] * 60 + [32] * 300,
    "every second": [200, 40] * 150,
    "few points": list(range(3, 18)) * 3,
}


@pytest.mark.parametrize("name", CASES)
def test_force(name):
    import torch
    import paper_2606_25569_amd as V
    sizes = CASES[name]
    X, off = _curves(sizes, 51)
    sigma = np.random.default_rng(8).normal(size=X.shape[1])
    for tension in (sigma, None):
        ref_f, ref_w = _centred_reference(X, np.zeros_like(sigma) if tension is None else tension, 0.9, off)
        f, w = V.elastic_force(torch.tensor(X, device="cuda"), off, 0.9,
                               None if tension is None else torch.tensor(tension, device="cuda"))
        f, w = f.cpu().numpy(), w.cpu().numpy()
        worst = 0.0
        for v, n in enumerate(sizes):
            a, b = off[v], off[v + 1]
            if n < 3:
                assert not np.isfinite(f[:, a:b]).any()
                continue
            ext = np.abs(X[:, a:b] - X[:, a:a + 1]).max()
            tol = 64 * EPS * ext * (n / 2) ** 4 + 64 * EPS * np.abs(ref_f[:, a:b]).max()
            tol_w = 16 * EPS * ext * n * max(1.0, np.log2(n)) * (2 * np.pi / n)
            worst = max(worst, np.abs(f[:, a:b] - ref_f[:, a:b]).max() / tol, np.abs(w[a:b] - ref_w[a:b]).max() / tol_w)
        say(f"{name}: force {worst:.3f} of the bound")
        assert worst <= 1.0


@pytest.mark.parametrize("name", CASES)
def test_layers(name):
    import torch
    import paper_2606_25569_amd as V
    sizes = CASES[name]
    X, w, off = weighted_curves(sizes, 52, clockwise=(2, 301))
    ref, _ = NR.near_layers(X, w, off)
    got = V.near_layers(torch.tensor(X, device="cuda"), torch.tensor(w, device="cuda"), off).cpu().numpy()
    worst = 0.0
    for v, n in enumerate(sizes):
        a, b = off[v], off[v + 1]
        g = got[:, 5 * a:5 * b]
        if n < 3:
            assert np.isnan(g).all()
            continue
        worst = max(worst, np.abs(g - ref[:, 5 * a:5 * b]).max() / _layer_tol(X[:, a:b], w[a:b], n))
    say(f"{name}: layers {worst:.3f} of the bound")
    assert worst <= 1.0


@pytest.mark.parametrize("name", ["small", "two wavefronts"])
def test_points_that_are_not_finite_stay_in_their_vesicle(name):
    import torch
    import paper_2606_25569_amd as V
    sizes = CASES[name]
    X, off = _curves(sizes, 53)
    good_f, good_w = V.elastic_force(torch.tensor(X, device="cuda"), off, 1.0, None)
    hit = [v for v in (0, 13, 501, len(sizes) - 1) if sizes[v] >= 3]
    for v in hit:
        X[0, off[v] + 1] = np.nan
    f, w = V.elastic_force(torch.tensor(X, device="cuda"), off, 1.0, None)
    for v in hit:
        a, b = off[v], off[v + 1]
        assert torch.isnan(f[:, a:b]).all() and not torch.isfinite(w[a:b]).any()
        f[:, a:b], w[a:b] = good_f[:, a:b], good_w[a:b]
    assert torch.equal(torch.nan_to_num(f), torch.nan_to_num(good_f))
    assert torch.equal(w, good_w)
