"""The float64 symmetric form at the edges of its work split: point counts around the blocks, strips and ring
cycles, vesicles that straddle them, and inputs that are not finite.  Bar as in test_gpu_symmetric64.py."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.gpu_util import dev_inputs, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu

BAR = 1e-12


@pytest.fixture(scope="module")
def V():
    import paper_2606_25569_amd as V
    return V


def _sizes(total, seed):
    """Vesicle sizes 0 .. 70 that add up to total."""
    rng = np.random.default_rng(seed)
    sizes = []
    while sum(sizes) < total:
        sizes.append(min(int(rng.integers(0, 71)), total - sum(sizes)))
    return sizes


def _run(V, s, config):
    import torch
    X, f, w = dev_inputs(s)
    out = V.farfield_forward(X, X, f, w, s.offsets, s.mu, precision="fp64", config=config)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("total", [31, 256, 257, 1023, 1040, 4095, 4096, 4097, 9217])
def test_point_counts_around_blocks_and_strips(V, total):
    """Every targets-per-thread and the automatic choice (direct below 4096 points)."""
    s = _ragged_suspension(seed=total, sizes=_sizes(total, total), spacing=4.5)
    ref = O.farfield_suspension(s.X, s.f, s.w, s.offsets, s.mu)
    for cfg in [None] + [{"pair_form": 2, "targets_per_thread": T} for T in (1, 2, 3, 4)]:
        err = float(np.abs(_run(V, s, cfg) - ref).max())
        say(f"float64 symmetric P={total} {cfg}: {err:.3e}")
        assert err <= BAR * np.abs(ref).max()  # zero for a single vesicle


@pytest.mark.parametrize("what", ["force", "point", "coincident"])
def test_not_finite_inputs_reach_the_outputs(V, what):
    """A NaN force or coordinate, and two coincident points of different vesicles, as in the direct form: no
    output that they enter is finite."""
    s = _ragged_suspension(seed=11, sizes=_sizes(4500, 5), spacing=4.5)
    own = np.repeat(np.arange(s.n_vesicles), np.diff(s.offsets))
    j = 2100
    hit = own != own[j]
    if what == "force":
        s.f[0, j] = np.nan
    elif what == "point":
        s.X[1, j] = np.nan
    else:
        k = int(np.flatnonzero(hit)[700])
        s.X[:, j] = s.X[:, k]
        hit = np.isin(np.arange(s.n_points), [j, k])
    out = _run(V, s, {"pair_form": 2})
    direct = _run(V, s, {"pair_form": 1})
    assert not np.isfinite(direct[:, hit]).any()
    assert not np.isfinite(out[:, hit]).any()
    if what == "coincident":
        assert np.isfinite(out[:, ~hit]).all()
