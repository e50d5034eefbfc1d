"""The compensated symmetric form's one-launch preparation (up to 1,024 vesicles) against the separate preparation and
evaluation entry points, bit for bit: empty vesicles, vesicles longer than a wavefront, both sides of its limit; and the
adjoint at that limit against the gathers."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import dev_inputs, rel_err, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [0, 1, 3])
@pytest.mark.parametrize("sizes", [[1, 1], [0, 5, 0, 700, 64, 65, 0], [40] * 30, [7] * 1024, [7] * 1025])
def test_equals_prepared(sizes, T):
    import torch
    import paper_2606_25569_amd as V
    from paper_2606_25569_amd import _lib as L
    s = _ragged_suspension(seed=len(sizes), sizes=sizes, spacing=4.5)
    X, f, w = dev_inputs(s)
    cfg = L.TileConfig.from_dict({"pair_form": 2, "targets_per_thread": T})
    one = V.farfield_forward(X, X, f, w, s.offsets, s.mu, "fp32c", config=cfg)
    lib, part = L.lib(), V.Partition(s.offsets)
    P, M, ref = part.n_points, part.n_vesicles, ctypes.byref(cfg)
    ws = torch.empty(lib.vesnet_farfield_workspace_bytes(P, M, 1, ref), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(X)
    p = lambda t: t.data_ptr()  # noqa: E731
    st = torch.cuda.current_stream().cuda_stream
    L.check(lib.vesnet_farfield_prepare(p(X), p(f), p(w), p(part.device), M, P, 1, p(ws), ws.numel(), st))
    L.check(lib.vesnet_farfield_evaluate(p(X), p(part.device), M, P, s.mu, p(out), 1, ref, p(ws), ws.numel(), st))
    assert torch.equal(one, out)


@pytest.mark.parametrize("vesicles", [1024, 1025])
def test_adjoint_at_the_limit(vesicles):
    import torch
    from paper_2606_25569_amd.farfield import farfield_backward, farfield_backward_points
    sizes = list(np.random.default_rng(vesicles).integers(0, 12, size=vesicles))
    s = _ragged_suspension(seed=3, sizes=sizes, spacing=4.5)
    X, f, w = dev_inputs(s)
    g = torch.tensor(np.random.default_rng(5).normal(size=X.shape), device="cuda")
    got = farfield_backward_points(X, f, w, s.offsets, s.mu, g, "fp32c")
    gt, gs, gf, gw = farfield_backward(X, X.clone(), f, w, s.offsets, s.mu, g, "fp64")
    for name, a, b in zip(("points", "force", "weights"), got, (gt + gs, gf, gw)):
        err = rel_err(a.cpu().numpy(), b.cpu().numpy())[0]
        say(f"adjoint M={vesicles} {name}: {err:.2e}")
        assert err <= 1e-5
