"""The one-launch float64 adjoint of small point arrays against the gathers on separate arrays (whose target and source
gradients are added), within the float64 bar, at the edges of its tiles and of its range; some gradients only, empty
vesicles, one vesicle."""
import numpy as np
import pytest

from tests.gpu_util import dev_inputs, rel_err, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


def _sizes(total):
    rng = np.random.default_rng(total)
    sizes = [0]
    while sum(sizes) < total:
        sizes.append(min(int(rng.integers(1, 130)), total - sum(sizes)))
    return sizes


@pytest.mark.parametrize("sizes", [[1], [40], [1, 1], [5, 0, 3], [63, 1, 64, 65]] +
                         [_sizes(n) for n in (1023, 1024, 1025, 2047, 2048, 2049)])
def test_against_gathers(sizes):
    import torch
    from paper_2606_25569_amd.farfield import farfield_backward, farfield_backward_points
    s = _ragged_suspension(seed=len(sizes), sizes=sizes, spacing=4.5)
    X, f, w = dev_inputs(s)
    g = torch.tensor(np.random.default_rng(5).normal(size=X.shape), device="cuda")
    got = farfield_backward_points(X, f, w, s.offsets, s.mu, g, "fp64")
    gt, gs, gf, gw = farfield_backward(X, X.clone(), f, w, s.offsets, s.mu, g, "fp64")
    for name, a, b in zip(("points", "force", "weights"), got, (gt + gs, gf, gw)):
        if len([n for n in sizes if n]) < 2:
            assert (a == 0).all()
            continue
        err = rel_err(a.cpu().numpy(), b.cpu().numpy())[0]
        say(f"adjoint P={s.n_points} {name}: {err:.2e}")
        assert err <= 1e-12
    if s.n_points > 2048:
        return  # the symmetric form, whose atomics add in no fixed order
    for need in ((True, False, False), (False, True, False), (False, False, True)):
        some = farfield_backward_points(X, f, w, s.offsets, s.mu, g, "fp64", need)
        for n, a, b in zip(need, some, got):
            assert (a is None) if not n else torch.equal(a, b)
