"""Layers of few channels on both sides of the rule between conv_smallc.hip and conv_rag.hip, ragged layers whose rows take more than half of the
LDS or whose outputs fit one channel tile, and formats per channel in the ragged kernels: against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)
from test_gpu_ragged import _case

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W    C    K   R  S  st pad
    (2, 11, 9, 4, 40, 3, 3, 1, 1),               # a first layer's channels
    (2, 11, 9, 5, 40, 3, 3, 1, 1),
    (4, 17, 16, 10, 70, 3, 3, 2, 1),             # 30 bytes of a kernel row
    (3, 9, 12, 31, 33, 1, 1, 1, 0),
    (50, 33, 25, 6, 9, 5, 5, 1, 2),
    (120, 33, 31, 7, 130, 1, 1, 1, 0),           # many tiles
    (1, 30, 51, 181, 48, 3, 3, 1, 1),            # rows of 84 KB
    (3, 15, 23, 250, 11, 5, 5, 1, 2),
    (40, 27, 59, 88, 22, 3, 3, 1, 1),            # outputs of one tile
    (30, 13, 15, 83, 131, 3, 3, 1, 1),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_small_channels(B, shape):
    N, H, W, C, K, R, S, st, pad = shape
    rng = np.random.default_rng(sum(shape))
    x, w, b = _case(rng, shape + (1,))
    shift = max(1, int(np.log2(np.sqrt(R * S * C) * 70 * 70 / 40)))
    xd, wd, bd = dev(x), dev(w), dev(b)
    y_ref, acc_ref = orc.conv_q(x, w, b, 4, shift, 4, st, pad, 1, True, want_acc=True)
    assert np.array_equal(host(B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, 1, True)[0]), y_ref)
    y, acc = B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, 1, True, want_acc=True)
    assert np.array_equal(host(y), y_ref) and np.array_equal(host(acc), acc_ref)
    for lo, hi in ((-4, shift + 2), (shift - 1, 24)):        # inside the range of the packed rounding, from 0 on, and outside it
        f_w = rng.integers(lo, hi, K).astype(np.int32)
        f_w[:2] = lo, hi - 1
        y, _ = B.conv_q_pc(xd, wd, bd, 4, dev(f_w), 0, st, pad, 1, False)
        assert np.array_equal(host(y), orc.conv_q(x, w, b, 4, f_w, 0, st, pad, 1, False)[0])
