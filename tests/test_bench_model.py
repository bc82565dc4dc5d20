"""The byte counts by which bench.py prices the row kernels of the materialised path."""
from __future__ import annotations

import pytest

import synth_inputs as S


def test_bytes_of_the_row_kernels():
    import bench
    c = S.custom_config(B=128, beam=10, V=8192, H=640, P=640, E=640, D=1024, prec="bf16", algo="aes", pred="stateless", ctx=2)
    M, K = 1280, 10
    few, lists, rows = (bench.kernel_bytes(n, c, M, 128, 250, K, 750) for n in ("k_utt_few", "k_utt_select", "k_row_select"))
    # 256 statistics of 8 bytes per row, 20 chunks per utterance, activations read and written, tables and frames, state and tree
    assert few == pytest.approx(M * 2048 + 128 * 20 * 128 + M * 640 * (2 + 12 + 2) + 4 * 640 + M * 76)
    assert lists - few == pytest.approx((M - 128) * 20 * 128)  # 20 chunks per row
    assert rows - lists == pytest.approx(M * 92)  # lists through memory
    assert bench.kernel_bytes("k_row_select", dict(c, lm=dict(order=2)), M, 128, 250, K, 750) - rows == pytest.approx(M * (8 * 8192 - 2048 - 20 * 128))
