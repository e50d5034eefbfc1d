"""The compensated symmetric form's own preparation at the edges of its steps of 256 points per wavefront and of the rule
that leaves few large vesicles to the separate kernels (2,048 points per vesicle on average): the same float32 sums
either way, against the oracle (1e-5 of the largest value, as in test_gpu_symmetric.py), and the adjoint with them."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.gpu_util import dev_inputs, rel_err, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[255, 256, 257], [1, 511, 0, 512, 513, 16], [2048, 2048], [2049, 2048], [4096, 3, 1],
                                   [1030, 17] * 3])
def test_sizes(sizes):
    import paper_2606_25569_amd as V
    s = _ragged_suspension(seed=sum(sizes), sizes=sizes, spacing=3.5)
    X, f, w = dev_inputs(s)
    ref = O.farfield_suspension(s.X, s.f, s.w, s.offsets, s.mu)
    u = V.farfield_forward(X, X, f, w, s.offsets, s.mu, "fp32c", config=dict(pair_form=2, targets_per_thread=1))
    err = rel_err(u.cpu().numpy(), ref)[0]
    g = np.random.default_rng(1).standard_normal(s.X.shape)
    want = O.grad_suspension(s.X, s.f, s.w, s.offsets, s.mu, g)
    got = V.farfield_backward_points(X, f, w, s.offsets, s.mu, X.new_tensor(g), "fp32c")
    errs = [rel_err(a.cpu().numpy(), b)[0] for a, b in zip(got, (want["grad_X"], want["grad_f"], want["grad_w"]))]
    say(f"{sizes}: forward {err:.1e}, gradients {errs}")
    assert err <= 1e-5 and max(errs) <= 1e-5
