"""Membrane force and near layers on many vesicles, where a workgroup takes several: one wavefront each for those of
up to 128 points, the whole workgroup for the larger ones among them, and none for empty or too large ones.  Bars are
those of test_gpu_spectral.py and test_gpu_rbf.py."""
import numpy as np
import pytest

from oracle import nearfield_rbf as NR
from tests.gpu_util import say
from tests.test_gpu_rbf import _curves as weighted_curves
from tests.test_gpu_rbf import _layer_tol
from tests.test_gpu_spectral import _check_force, _curves, _exact_shift

pytestmark = pytest.mark.gpu


def _sizes(seed):
    """1,300 vesicles (six to a workgroup) at the edges of the 16-point blocks and of the two forms."""
    rng = np.random.default_rng(seed)
    sizes = rng.choice([1, 2, 3, 5, 15, 16, 17, 31, 32, 33, 48, 65, 112, 113, 127, 128], 1300)
    sizes[[7, 300, 301]] = [129, 400, 144]
    sizes[[501, 502, 1299]] = [1024, 0, 257]
    return [int(n) for n in sizes]


@pytest.mark.parametrize("shift", [0.0, 1000.0])
def test_force(shift):
    import paper_2606_25569_amd as V
    sizes = _sizes(3)
    X, off = _curves(sizes, 41)
    _, X1 = _exact_shift(X, off, shift)
    sigma = np.random.default_rng(8).normal(size=X.shape[1])
    _check_force(V, X1, off, sizes, sigma, 0.9, f"blocks +{shift:g}")


def test_layers():
    import torch
    import paper_2606_25569_amd as V
    sizes = _sizes(4)
    X, w, off = weighted_curves(sizes, 42, clockwise=(2, 301))
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
    say(f"layers: worst error {worst:.3f} of the bound")
    assert worst <= 1.0


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_not_finite_points_stay_in_their_vesicle(bad):
    import torch
    import paper_2606_25569_amd as V
    sizes = _sizes(5)
    X, off = _curves(sizes, 43)
    good_f, good_w = V.elastic_force(torch.tensor(X, device="cuda"), off, 1.0, None)
    hit = [v for v in (10, 300, 700) if sizes[v] >= 3]
    for v in hit:
        X[0, off[v] + 1] = bad
    f, w = V.elastic_force(torch.tensor(X, device="cuda"), off, 1.0, None)
    for v in hit:
        a, b = off[v], off[v + 1]
        assert torch.isnan(f[:, a:b]).all() and not torch.isfinite(w[a:b]).any()
        f[:, a:b], w[a:b] = good_f[:, a:b], good_w[a:b]
    assert torch.equal(torch.nan_to_num(f), torch.nan_to_num(good_f))
    assert torch.equal(w, good_w)
