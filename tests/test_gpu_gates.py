"""The divisions of the LSTM cell (device_utils.h: sigmoid_of, tanh_of) against IEEE float32 division, bit for bit, over every exponent that
their argument can have."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_gates_are_the_correctly_rounded_quotients():
    import torch
    import paper_2506_00185_amd.binding as Bd
    rng = np.random.default_rng(1)
    mant = np.concatenate([[0, 1, 2, (1 << 23) - 2, (1 << 23) - 1], rng.integers(0, 1 << 23, 2043)])
    e = (np.arange(255)[:, None] << 23 | mant[None, :]).astype(np.uint32).ravel().view(np.float32)  # 0 to the largest finite one
    near_one = (np.float32(1).view(np.uint32) - np.arange(4096, dtype=np.uint32)).view(np.float32)
    e = np.concatenate([e, near_one, [np.float32(np.inf)]]).astype(np.float32)
    sig, tanh = (t.cpu().numpy() for t in Bd.debug_gates(torch.as_tensor(e).cuda()))
    one = np.float32(1)
    with np.errstate(all="ignore"):
        want_sig, want_tanh = one / (one + e), (one - e) / (one + e)
    assert want_sig[(e > 2.0 ** 126) & (e < np.inf)].min() > 0  # subnormal, not 0
    np.testing.assert_array_equal(sig.view(np.uint32), want_sig.view(np.uint32))
    np.testing.assert_array_equal(tanh[e <= 1].view(np.uint32), want_tanh[e <= 1].view(np.uint32))
    bad = Bd.debug_gates(torch.full((3,), float("nan"), device="cuda"))
    assert all(torch.isnan(x).all() for x in bad)
