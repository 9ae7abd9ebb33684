"""The dense kernel in steps of 128 bytes against the oracle: every tile shape on both sides of its line, ragged pixel tiles,
strides, padding and one weight format per output channel."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_ops import B, _ties_bias, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W    C    K   R  S  st pad
    (3, 40, 41, 128, 128, 3, 3, 1, 1),           # 64 x 64
    (2, 31, 33, 256, 192, 1, 1, 1, 0),           # 64 x 64, K no multiple of 128
    (11, 57, 59, 128, 64, 3, 3, 2, 1),
    (1, 67, 70, 128, 320, 5, 3, 1, 3),           # padding beyond the kernel's half
    (20, 43, 41, 128, 64, 1, 1, 1, 0),           # 128 x 64, one step
    (24, 43, 41, 256, 64, 3, 3, 1, 1),
    (9, 53, 55, 128, 128, 3, 3, 1, 1),           # 128 x 128, eight wavefronts
    (16, 29, 30, 384, 384, 1, 1, 2, 0),
    (13, 45, 43, 512, 128, 1, 1, 1, 0),          # 128 x 128, four wavefronts
    (40, 31, 29, 128, 256, 3, 3, 1, 1),          # 256 x 256, 141 tiles
    (40, 61, 57, 128, 256, 3, 3, 2, 1),
    (47, 21, 19, 1024, 512, 1, 1, 1, 0),         # two channel tiles
    (26, 30, 32, 128, 384, 1, 1, 1, 0),          # 128 x 64 for a little more than one round of 128 x 128
    (27, 30, 30, 128, 384, 3, 3, 1, 1),
    (25, 14, 14, 256, 1024, 1, 1, 1, 0),         # 128 x 128, four wavefronts, a short chain
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_wide_steps(B, shape):
    N, H, W, C, K, R, S, st, pad = shape
    rng = np.random.default_rng(sum(shape))
    x, w = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (K, R, S, C)).astype(np.int8)
    b = rng.integers(-2 ** 15, 2 ** 15, (K,)).astype(np.int32)
    xd, wd, bd = dev(x), dev(w), dev(b)
    shift = int(np.log2(np.sqrt(R * S * C) * 70 * 70 / 40))
    y_ref, _ = orc.conv_q(x, w, b, 4, shift, 4, st, pad, 1, True)
    assert np.array_equal(host(B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, 1, True)[0]), y_ref)
    # without bias and ReLU, into a channel slice of a wider tensor
    y_ref, _ = orc.conv_q(x, w, None, 4, shift - 2, 4, st, pad, 1, False)
    wide = torch.full((N, y_ref.shape[1], y_ref.shape[2], K + 32), 77, dtype=torch.int8, device="cuda")
    B.conv_q(xd, wd, None, 4, shift - 2, 4, st, pad, 1, False, out=wide.view(-1)[16:], ldy=K + 32)
    got = host(wide)
    assert np.array_equal(got[..., 16:16 + K], y_ref)
    assert (got[..., :16] == 77).all() and (got[..., 16 + K:] == 77).all()
    # one weight format per output channel
    f_w = rng.integers(shift - 3, shift + 2, K).astype(np.int32)
    y_ref, _ = orc.conv_q(x, w, b, 4, f_w, 4, st, pad, 1, False)
    assert np.array_equal(host(B.conv_q_pc(xd, wd, bd, 4, dev(f_w), 4, st, pad, 1, False)[0]), y_ref)


@pytest.mark.parametrize("s", [0, 1, 22, 23, 24])
@pytest.mark.parametrize("shape", [(2, 31, 33, 256, 192, 1, 1),          # steps of 128 bytes: 64 x 64
                                   (20, 43, 41, 128, 64, 1, 1),          # 128 x 64
                                   (26, 30, 32, 128, 384, 1, 1),
                                   (13, 45, 43, 512, 128, 1, 1),         # 128 x 128, four wavefronts
                                   (9, 53, 55, 128, 128, 3, 1),          # eight
                                   (40, 31, 29, 128, 256, 3, 1),         # 256 x 256
                                   (1, 30, 30, 64, 128, 3, 1),           # steps of 64 bytes: 64 x 64
                                   (5, 30, 30, 192, 128, 1, 1),          # 128 x 128
                                   (38, 30, 30, 64, 128, 3, 1),          # 256 x 128
                                   (55, 30, 30, 64, 256, 1, 1),          # 256 x 256
                                   (3, 30, 30, 192, 64, 3, 1)],          # 256 x 64
                         ids=lambda s: "x".join(map(str, s)))
def test_rounding_at_the_edges_of_the_lean_range(B, shape, s):
    """Every tile shape of the dense kernel, by name, at the smallest and largest shifts of the four-instruction rounding and at the
    first one behind it; biases are ties and near-ties of the shift, and small operands leave the results unsaturated."""
    N, H, W, C, K, R, st = shape
    rng = np.random.default_rng(sum(shape) + s)
    x, w = rng.integers(-1, 2, (N, H, W, C)).astype(np.int8), rng.integers(-1, 2, (K, R, R, C)).astype(np.int8)
    b = _ties_bias(rng, K, s)
    f_in, f_w = 6, 12
    f_out = f_in + f_w - s
    ref, _ = orc.conv_q(x, w, b, f_in, f_w, f_out, st, R // 2, 1, False)
    assert (np.abs(ref) == 127).mean() < 0.5
    got, _ = B.conv_q(dev(x), dev(w), dev(b), f_in, f_w, f_out, st, R // 2, 1, False, variant=B.CONV_MFMA)
    assert np.array_equal(host(got), ref)
    # one weight format per output channel, shifts up to s
    sk = rng.integers(max(0, s - 3), s + 1, K)
    sk[:2] = (max(0, s - 3), s)
    f_wk = (f_out - f_in + sk).astype(np.int32)
    bk = np.array([_ties_bias(rng, 1, int(v))[0] for v in sk], np.int32)
    ref, _ = orc.conv_q(x, w, bk, f_in, f_wk, f_out, st, R // 2, 1, True)
    got, _ = B.conv_q_pc(dev(x), dev(w), dev(bk), f_in, dev(f_wk), f_out, st, R // 2, 1, True)
    assert np.array_equal(host(got), ref)
