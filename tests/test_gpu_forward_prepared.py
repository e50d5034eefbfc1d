"""vesnet_farfield_stokeslet is prepare + evaluate: whatever launches it takes, its workspace holds the prepared region
afterwards, and vesnet_farfield_evaluate at a second set of targets gives what it gives after vesnet_farfield_prepare,
bit for bit.  Sizes on every route: one launch (float64 of 4, 8 and 16 targets to a workgroup; compensated), the
symmetric form that prepares itself, three launches, and vesicles without points."""
import ctypes

import pytest

from tests.gpu_util import dev_inputs
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu

SYM = dict(pair_form=2, targets_per_thread=1)


@pytest.mark.parametrize("precision,sizes,config", [
    ("fp32c", [32] * 16, None), ("fp32c", [1, 0, 70, 33, 5], None), ("fp32c", [32] * 33, None),
    ("fp32c", [32] * 504, None), ("fp32c", [32, 0, 17, 300] * 12, SYM), ("fp32c", [3] * 1030, SYM),
    ("fp64", [32] * 16, None), ("fp64", [32] * 48, None), ("fp64", [1, 0, 700, 33, 2000], None), ("fp64", [4] * 1024, None),
    ("fp64", [41] * 100, None), ("fp64", [32] * 20, SYM), ("fp32", [32] * 16, None)])
def test_evaluate_after_the_call(precision, sizes, config):
    import torch
    from paper_2606_25569_amd import Partition, _lib as L
    from paper_2606_25569_amd.farfield import workspace_bytes
    s = _ragged_suspension(seed=len(sizes), sizes=sizes, spacing=3.5)
    X, f, w = dev_inputs(s)
    part = Partition(s.offsets)
    P, M, prec = part.n_points, part.n_vesicles, L.precision_code(precision)
    cfg = ctypes.byref(L.TileConfig.from_dict(config)) if config else None
    st = torch.cuda.current_stream().cuda_stream
    lib = L.lib()
    Y = X if config else (X + 0.01).contiguous()  # the symmetric form takes the prepared points as its targets
    got = []
    for whole in (True, False):
        ws = torch.full((workspace_bytes(P, M, precision, config),), 255, dtype=torch.uint8, device="cuda")
        u, v = torch.empty_like(X), torch.empty_like(X)
        src = (X.data_ptr(), f.data_ptr(), w.data_ptr(), part.device.data_ptr(), M, P)
        if whole:
            L.check(lib.vesnet_farfield_stokeslet(X.data_ptr(), *src, 0.7, u.data_ptr(), prec, cfg, ws.data_ptr(),
                                                  ws.numel(), st))
        else:
            L.check(lib.vesnet_farfield_prepare(*src, prec, ws.data_ptr(), ws.numel(), st))
        L.check(lib.vesnet_farfield_evaluate(Y.data_ptr(), part.device.data_ptr(), M, P, 0.7, v.data_ptr(), prec, cfg,
                                             ws.data_ptr(), ws.numel(), st))
        got.append(v)
    assert torch.isfinite(got[1]).all()
    assert torch.equal(*got)
