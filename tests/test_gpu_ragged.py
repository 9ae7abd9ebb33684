"""The matrix-core kernel for any number of channels (conv_rag.hip) against the oracle, at the edges of its segments, tiles and
loads, with operands and results at odd addresses."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W    C    K   R  S  st pad groups
    (1, 1, 1, 16, 1, 1, 1, 1, 0, 1),             # one piece, one output
    (1, 3, 16, 1, 40, 1, 1, 1, 0, 1),            # a row of exactly one piece
    (2, 5, 7, 5, 9, 3, 3, 1, 1, 1),              # the kernel row is shorter than a piece
    (1, 9, 8, 16, 65, 3, 3, 1, 1, 1),            # whole pieces, channel tile + 1
    (2, 9, 7, 17, 64, 3, 3, 2, 1, 1),            # one byte over a piece
    (1, 6, 5, 43, 63, 5, 5, 1, 2, 1),            # padding wider than a step on the left and the right
    (3, 13, 11, 83, 131, 3, 3, 1, 1, 1),
    (1, 33, 4, 21, 33, 3, 3, 1, 2, 1),           # outputs wholly in the padding's reach
    (1, 40, 40, 37, 70, 4, 2, 3, 1, 1),          # even kernel, stride 3
    (1, 70, 6, 3, 10, 35, 3, 1, 17, 1),          # more kernel rows than the other kernels' masks hold
    (2, 64, 64, 7, 130, 3, 3, 1, 1, 1),          # enough tiles for the 128-pixel form
    (17, 64, 62, 30, 72, 3, 3, 1, 1, 1),
    (2, 9, 11, 30, 40, 3, 3, 1, 1, 2),           # groups of 15 -> 20
    (1, 10, 9, 99, 27, 3, 3, 2, 1, 3),           # groups of 33 -> 9
    (1, 7, 7, 130, 200, 3, 3, 1, 1, 2),          # groups of 65 -> 100: several channel tiles per group
    (2, 8, 9, 51, 34, 1, 1, 1, 0, 17),           # groups of 3 -> 2
    (1, 12, 10, 25, 25, 5, 3, 2, 2, 25),         # one channel per group
]


def _case(rng, shape):
    N, H, W, C, K, R, S, st, pad, g = shape
    return (rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (K, R, S, C // g)).astype(np.int8),
            rng.integers(-2 ** 15, 2 ** 15, (K,)).astype(np.int32))


def _odd(a, off):
    """A device copy of `a` that starts `off` bytes into an allocation."""
    buf = torch.zeros(a.nbytes + 64, dtype=torch.int8, device="cuda")
    v = buf[off:off + a.nbytes].view(a.shape)
    v.copy_(dev(a))
    return v


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_ragged(B, shape):
    N, H, W, C, K, R, S, st, pad, g = shape
    rng = np.random.default_rng(sum(shape))
    x, w, b = _case(rng, shape)
    shift = max(0, int(np.log2(np.sqrt(R * S * (C // g)) * 70 * 70 / 40)))
    for i, (relu, bias, s) in enumerate([(True, True, shift), (False, False, shift - 2), (True, True, 24)]):
        f_in, f_w, f_out = 4, s, 4
        y_ref, acc_ref = orc.conv_q(x, w, b if bias else None, f_in, f_w, f_out, st, pad, g, relu, want_acc=True)
        y, acc = B.conv_q(dev(x), dev(w), dev(b) if bias else None, f_in, f_w, f_out, st, pad, g, relu, want_acc=i == 0, variant=B.CONV_RAGGED)
        assert np.array_equal(host(y), y_ref), (relu, bias, s)
        if i == 0:
            assert np.array_equal(host(acc), acc_ref)
    # every operand at an odd address, the result in a channel slice of a wider tensor with an odd pitch
    ldy = K + 6
    wide = torch.full((N, y_ref.shape[1], y_ref.shape[2], ldy), 77, dtype=torch.int8, device="cuda")
    y_ref, _ = orc.conv_q(x, w, b, 4, shift, 4, st, pad, g, True)
    B.conv_q(_odd(x, 3), _odd(w, 5), dev(b), 4, shift, 4, st, pad, g, True, out=wide.view(-1)[1:], ldy=ldy, variant=B.CONV_RAGGED)
    got = host(wide).reshape(-1, ldy)
    assert np.array_equal(got[:, 1:1 + K], y_ref.reshape(-1, K))
    assert (got[:, 0] == 77).all() and (got[:, 1 + K:] == 77).all()
    # one weight format per output channel
    f_w = rng.integers(max(0, shift - 3), shift + 2, K).astype(np.int32)
    y_ref, _ = orc.conv_q(x, w, b, 4, f_w, 4, st, pad, g, False)
    y, _ = B.conv_q_pc(dev(x), dev(w), dev(b), 4, dev(f_w), 4, st, pad, g, False)
    assert np.array_equal(host(y), y_ref)


def test_batch_beyond_31_bit_offsets(B):
    """2.3 GB of input: the batch is cut into launches whose byte offsets fit 31 bits.  Result in a channel slice of a wider tensor and
    accumulators, against calls of a few images on both sides of the cut and at the ends."""
    N, H, C, K = 17200, 64, 33, 5
    most = (2 ** 31 - 1 - (1 + 3) * H * C) // (H * H * C)               # images of the first launch
    assert most < N
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(-128, 128, (N, H, H, C), dtype=torch.int8, device="cuda", generator=gen)
    w = torch.randint(-128, 128, (K, 3, 3, C), dtype=torch.int8, device="cuda", generator=gen)
    b = torch.randint(-10000, 10001, (K,), dtype=torch.int32, device="cuda", generator=gen)
    wide = torch.full((N, 32, 32, K + 3), 77, dtype=torch.int8, device="cuda")
    acc = torch.empty((N, 32, 32, K), dtype=torch.int32, device="cuda")
    B.conv_q(x, w, b, 4, 13, 4, 2, 1, 1, False, out=wide.view(-1)[2:], ldy=K + 3, acc_out=acc, variant=B.CONV_RAGGED)
    for first in (0, most - 2, most, N - 3):
        part = slice(first, first + 3)
        y_ref, acc_ref = orc.conv_q(host(x[part]), host(w), host(b), 4, 13, 4, 2, 1, 1, False, want_acc=True)
        assert np.array_equal(host(acc[part]), acc_ref), first
        assert np.array_equal(host(wide[part])[..., 2:2 + K], y_ref), first
    assert bool((wide[..., :2] == 77).all()) and bool((wide[..., 2 + K:] == 77).all())
