"""Column strips of the compensated symmetric form end at vesicle starts, so that every float32 partial sum is the one of
whole block pairs: a call that the launch rule cuts into strips agrees with the same call at the named targets per thread,
which it does not cut, up to the fixed-point roundings of the rows (one more per strip, half of 2^-S each, 2^S from the
bound 520 sum |F|) and the float64 sums before them.  A cut inside a vesicle would round its float32 sums differently,
about 1e-8 of sum |F|.  The two results differ in some bits, which shows that strips were taken."""
import math

import numpy as np
import pytest

from tests.gpu_util import dev_inputs, say
from tests.test_gpu_symmetric import _ragged_suspension

pytestmark = pytest.mark.gpu


# sizes, targets per thread and strips of the rule: whole vesicles per strip (512 x 64: two to a strip of eight cycles),
# and below 1,024 units strips of four cycles whatever the sizes, with vesicles longer than a strip and starting anywhere
@pytest.mark.parametrize("sizes,T,strips,config", [
    ([32] * 504, 1, 2, None), ([64] * 512, 2, 4, None), ([17, 63, 40] * 40, 1, 4, dict(pair_form=2)),
    ([100, 7, 300, 33, 1, 64] * 9, 1, 2, dict(pair_form=2)), ([48] * 60, 1, 4, dict(pair_form=2))])
def test_strips_leave_the_partial_sums(sizes, T, strips, config):
    import torch
    import paper_2606_25569_amd as V
    s = _ragged_suspension(seed=len(sizes), sizes=sizes, spacing=3.5)
    X, f, w = dev_inputs(s)
    cut = V.farfield_forward(X, X, f, w, s.offsets, s.mu, "fp32c", config=config)
    whole = V.farfield_forward(X, X, f, w, s.offsets, s.mu, "fp32c", config=dict(pair_form=2, targets_per_thread=T))
    total = float(np.abs(s.w * s.f).sum())
    cycles = sum(-(-n // 16) for n in sizes)
    blocks = -(-cycles // (16 * T))
    S = 62 - math.frexp(520.0 * total)[1]
    # rows: at most `blocks` units of `strips` roundings each; float64: at most 8 |F| per pair, half an ulp per addition
    tol = (2 * blocks * strips * 2.0**-S + 8 * total * 2.0**-52) / (4 * math.pi * s.mu)
    diff = float((cut - whole).abs().max())
    say(f"{len(sizes)} vesicles: difference {diff:.1e} of {tol:.1e}, max |u| {float(whole.abs().max()):.1e}")
    assert diff <= tol
    assert not torch.equal(cut, whole)
