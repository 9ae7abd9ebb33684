"""Convolutions into a channel slice whose tensor lies directly in front of another operand."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


def test_last_slice_with_the_input_right_behind_it(B):
    """The last row of a slice ends with its own channels: the bytes that ldy adds behind them are not touched, and may be the input's."""
    rng = np.random.default_rng(5)
    N, H, W, C, K, ldy = 2, 7, 9, 32, 16, 48
    x = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8)
    w = rng.integers(-128, 128, (K, 1, 1, C)).astype(np.int8)
    joined = N * H * W * ldy
    buf = torch.zeros(joined + x.nbytes, dtype=torch.int8, device="cuda")
    xd = buf[joined:].view(x.shape)
    xd.copy_(dev(x))
    y_ref, _ = orc.conv_q(x, w, None, 4, 7, 2, 1, 0, 1, True)
    B.conv_q(xd, dev(w), None, 4, 7, 2, relu=True, out=buf[ldy - K:], ldy=ldy)
    assert np.array_equal(host(buf[:joined]).reshape(-1, ldy)[:, ldy - K:], y_ref.reshape(-1, K))
    assert np.array_equal(host(xd), x)
    with pytest.raises(B.DfqError):                  # one byte further and the last row does reach into the input
        B.conv_q(xd, dev(w), None, 4, 7, 2, relu=True, out=buf[ldy - K + 1:], ldy=ldy)
