"""Column strips of the compensated symmetric kernels: strips end at vesicle starts, so the float32 partial sums,
and with them the result up to the fixed-point resolution, are those of whole block pairs."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.gpu_util import dev_inputs, rel_err, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import paper_2606_25569_amd as V
    return V


# points per vesicle and vesicles of problems that take two or four strips (and one whose long vesicles take none)
CASES = [("short vesicles, one target per thread", 17, 48, 380), ("medium, two targets", 40, 64, 640),
         ("long", 120, 130, 100), ("ragged with empty ones", 0, 70, 400)]


@pytest.mark.parametrize("name,lo,hi,m", CASES)
def test_forward_strips_keep_the_partial_sums(V, name, lo, hi, m):
    """The automatic choice (strips) against whole block pairs (an explicit targets_per_thread) within the
    fixed-point resolution, 2^-S per row partial with S at least 38 at these sizes: 1e-10 of max |u| covers the
    hundreds of partials of a point."""
    import torch
    sizes = [int(x) for x in np.random.default_rng(m).integers(lo, hi + 1, size=m)]
    s = _ragged_suspension(seed=m, sizes=sizes, spacing=4.5)
    X, f, w = dev_inputs(s)
    auto = V.farfield_forward(X, X, f, w, s.offsets, s.mu, precision="fp32c", config={"pair_form": 2})
    again = V.farfield_forward(X, X, f, w, s.offsets, s.mu, precision="fp32c", config={"pair_form": 2})
    assert torch.equal(auto, again)
    best = min(float((V.farfield_forward(X, X, f, w, s.offsets, s.mu, precision="fp32c",
                                         config={"pair_form": 2, "targets_per_thread": T}) - auto).abs().max())
               for T in (1, 2, 3))  # the automatic T is one of them
    scale = float(auto.abs().max())
    say(f"{name}: strips against whole pairs {best / scale:.3e}")
    assert best <= 1e-10 * scale


@pytest.mark.parametrize("sizes", [[32] * 128, [32] * 16, [130] * 20, [5] * 300, [700, 3, 0, 650, 40]])
def test_adjoint_strips_against_oracle(V, sizes):
    """Gradients at sizes that take one, two and four strips; 1e-5 as in test_gpu_adjoint_points.py."""
    import torch
    s = _ragged_suspension(seed=len(sizes), sizes=sizes, spacing=5.0)
    g = np.random.default_rng(3).normal(size=s.X.shape)
    X, f, w = dev_inputs(s)
    got = V.farfield_backward_points(X, f, w, s.offsets, s.mu, torch.tensor(g, device="cuda"), "fp32c")
    ref = O.grad_suspension(s.X, s.f, s.w, s.offsets, s.mu, g)
    for key, a in zip(("grad_X", "grad_f", "grad_w"), got):
        err = rel_err(a.cpu().numpy(), ref[key])[0]
        say(f"adjoint strips {len(sizes)} vesicles {key}: {err:.3e}")
        assert err <= 1e-5
