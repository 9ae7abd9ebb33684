"""The calibration maximum of (8, p) layers on the matrix cores (dfq_conv_np_absmax) where its tiles have edges, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle.npconv as NC

from test_gpu_npconv import B, dev               # noqa: F401  (B is a fixture)
from test_gpu_npnet import planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,C,K,R,stride,pad", [
    (1, 1, 1, 64, 16, 1, 1, 0),                  # one pixel: 127 rows of the tile are empty
    (2, 13, 5, 64, 80, 3, 1, 1),                 # 130 pixels, a second channel tile of 16
    (1, 9, 9, 192, 64, 3, 2, 1),
    (1, 6, 7, 320, 32, 3, 1, 1),                 # 45 steps: the three-stage form
])
@pytest.mark.parametrize("relu", [False, True])
def test_conv_np_absmax_tiles(B, N, H, W, C, K, R, stride, pad, relu):
    rng = np.random.default_rng(C + K)
    x = rng.integers(0, 256, (N, H, W, C)).astype(np.uint8)
    w = rng.integers(0, 256, (K, R, R, C)).astype(np.uint8)
    # channel 3 has a bias that its own sums nearly cancel: a tile row without a pixel would report the bias alone
    w[3] = 0x7f
    x[...] = np.where(rng.random(x.shape) < 0.5, 0xff, 0xf0)
    prod = NC.conv_sum(NC.decode_tensor(x, 8, 4), NC.decode_tensor(w, 8, 4), stride, pad, 1)
    b = rng.integers(-1000, 1000, K).astype(np.int32)
    b[3] = min(2 ** 31 - 1, int(-prod[..., 3].max()))
    acc = prod + b.astype(np.int64)
    want = int((np.maximum(acc, 0) if relu else np.abs(acc)).max())
    assert B.conv_np_absmax(*planes(B, x, 4), *planes(B, w, 4), dev(b), stride, pad, 1, relu) == want
