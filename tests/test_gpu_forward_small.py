"""The one-launch direct sums of small problems: the default call against the same sum in the prepared form (an explicit
launch shape), compensated bit for bit, float64 within its bar, at the edges of the tiles and of their ranges; empty
vesicles, one vesicle, vesicles of more than 64 points, separate target arrays."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import suspension as S
from tests.gpu_util import dev_inputs, rel_err, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu

BAR = {"fp64": 1e-12, "fp32c": 1e-5}


def _check(s, prec, moved, name):
    import torch
    import paper_2606_25569_amd as V
    X, f, w = dev_inputs(s)
    T = X + 0.01 * torch.sin(3 * X) if moved else X
    small = V.farfield_forward(T, X, f, w, s.offsets, s.mu, prec)
    prepared = V.farfield_forward(T, X, f, w, s.offsets, s.mu, prec, config={"pair_form": 1})
    assert torch.equal(small, V.farfield_forward(T, X, f, w, s.offsets, s.mu, prec))
    if prec == "fp32c":
        assert torch.equal(small, prepared)
    if int(np.sum(np.diff(s.offsets) > 0)) < 2:
        assert (small == 0).all()
        return
    assert rel_err(small.cpu().numpy(), prepared.cpu().numpy())[0] <= BAR["fp64"]
    if not moved:
        ref = O.farfield_suspension(s.X, s.f, s.w, s.offsets, s.mu)
        err, _ = rel_err(small.cpu().numpy(), ref)
        say(f"small {prec} {name} P={s.n_points}: {err:.2e}")
        assert err <= BAR[prec]


@pytest.mark.parametrize("moved", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32c"])
@pytest.mark.parametrize("sizes", [
    [1], [1, 1], [5, 0, 3], [63, 1, 64, 65], [129, 2, 31, 200, 0, 70], [32] * 16, [32] * 32, [31] * 33, [1000, 24],
    [1024, 0], [3] * 31 + [900]])
def test_sizes(prec, moved, sizes):
    _check(_ragged_suspension(seed=len(sizes), sizes=sizes, spacing=4.5), prec, moved, f"{len(sizes)} vesicles")


@pytest.mark.parametrize("total", [1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
def test_float64_tiles(total):
    rng = np.random.default_rng(total)
    sizes = []
    while sum(sizes) < total:
        sizes.append(min(int(rng.integers(1, 100)), total - sum(sizes)))
    s = _ragged_suspension(seed=total, sizes=sizes, spacing=4.5)
    _check(s, "fp64", True, "tiles")
    _check(s, "fp64", False, "tiles")
