"""Grouped layers taken several groups at a time (conv_rag_groups.hip) against the oracle: blocks that do not divide the groups, groups wider than a
block, one and several channels in a group, tiles that cross rows and images, both tile sizes, every form of the epilogue, odd addresses."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_dispatch import launched
from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)
from test_gpu_ragged import _case, _odd

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W    C    K   R  S  st pad groups
    (90, 7, 7, 99, 99, 3, 3, 1, 1, 33),          # groups of 3 -> 3: 10 to a block, 3 in the last; a tile crosses images
    (29, 13, 12, 97, 97, 3, 3, 1, 1, 97),        # one channel in a group
    (12, 9, 31, 126, 336, 3, 3, 2, 1, 42),       # groups of 3 -> 8, rows and columns skipped
    (3, 17, 15, 85, 80, 5, 5, 1, 2, 5),          # groups of 17 -> 16: two pieces and one byte
    (10, 23, 20, 96, 160, 5, 5, 1, 2, 4),        # groups of 24 -> 40: two blocks of one group
    (3000, 1, 1, 198, 198, 5, 5, 1, 2, 66),      # every pixel its own image, only the middle tap inside
    (60, 33, 31, 126, 126, 3, 1, 3, 0, 42),      # a kernel of one column, stride 3
    (20, 40, 9, 93, 155, 2, 4, 1, 3, 31),        # even kernels, outputs wholly in the padding
    (36, 30, 31, 224, 96, 3, 3, 2, 1, 32),       # 10 groups of 7 -> 3: five pieces
    (40, 33, 29, 80, 160, 3, 3, 1, 1, 16),       # 256 pixels to a workgroup, several tiles each
    (70, 29, 27, 70, 42, 3, 3, 1, 1, 14),
    (60, 40, 37, 24, 24, 1, 1, 1, 0, 12),
]
# several groups at a time but for sums, which go out one by one
CODES = [
    (40, 19, 23, 300, 120, 1, 1, 1, 0, 12),      # groups of 25 -> 10
    (3, 33, 130, 99, 99, 1, 3, 1, 1, 11),        # rows longer than a tile
    (9, 33, 31, 128, 264, 3, 3, 1, 1, 8),        # groups of 16 -> 33
]
# one group at a time
SMALL = [
    (17, 19, 23, 300, 124, 1, 1, 1, 0, 4),       # groups of 75 -> 31
    (700, 1, 1, 99, 99, 5, 5, 1, 2, 11),
    (60, 33, 31, 126, 90, 3, 1, 3, 0, 18),
    (12, 30, 31, 224, 96, 3, 3, 2, 1, 32),
    (9, 23, 20, 128, 264, 3, 3, 1, 1, 8),
    (11, 53, 16, 256, 256, 3, 3, 3, 0, 4),       # groups of 64, rows skipped
]


def test_kernels_of_the_shapes(B):
    """Which kernel the calls below reach, read from the device's records: these tests are about conv_rag_kernel_groups."""
    plain, sums, formats = [], [], []
    for N, H, W, C, K, R, S, st, pad, g in SHAPES + CODES + SMALL:
        x = torch.randint(-128, 128, (N, H, W, C), dtype=torch.int8, device="cuda")
        w = torch.randint(-128, 128, (K, R, S, C // g), dtype=torch.int8, device="cuda")
        f = torch.full((K,), 8, dtype=torch.int32, device="cuda")
        plain.append(lambda x=x, w=w, a=(st, pad, g): B.conv_q(x, w, None, 4, 8, 4, *a, True, variant=B.CONV_RAGGED))
        sums.append(lambda x=x, w=w, a=(st, pad, g): B.conv_q(x, w, None, 4, 8, 4, *a, True, want_acc=True, variant=B.CONV_RAGGED))
        formats.append(lambda x=x, w=w, f=f, a=(st, pad, g): B.conv_q_pc(x, w, None, 4, f, 4, *a, True, frac_w_range=(8, 8)))
    n, codes, small = len(SHAPES), len(CODES), len(SMALL)
    groups = lambda names: ["conv_rag_kernel_groups" in name for name in names]
    assert groups(launched(plain)) == [True] * (n + codes) + [False] * small
    assert groups(launched(sums)) == [True] * n + [False] * (codes + small)
    assert groups(launched(formats[:n + codes])) == [True] * (n + codes)


@pytest.mark.parametrize("shape", SHAPES + CODES + SMALL, ids=lambda s: "x".join(map(str, s)))
def test_conv_groups(B, shape):
    N, H, W, C, K, R, S, st, pad, g = shape
    rng = np.random.default_rng(sum(shape))
    x, w, b = _case(rng, shape)
    shift = max(1, int(np.log2(np.sqrt(R * S * (C // g)) * 70 * 70 / 40)))
    y_ref, acc_ref = orc.conv_q(x, w, b, 4, shift, 4, st, pad, g, True, want_acc=True)
    xd, wd, bd = dev(x), dev(w), dev(b)
    y, _ = B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, g, True, variant=B.CONV_RAGGED)
    assert np.array_equal(host(y), y_ref)
    assert np.array_equal(host(B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, g, True)[0]), y_ref)
    for want_y in (False, True):
        y, acc = B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, g, True, want_y=want_y, want_acc=True, variant=B.CONV_RAGGED)
        assert np.array_equal(host(acc), acc_ref) and (y is None or np.array_equal(host(y), y_ref))
    # no bias, and a shift beyond the four-instruction rounding
    y, _ = B.conv_q(xd, wd, None, 4, 25, 4, st, pad, g, False, variant=B.CONV_RAGGED)
    assert np.array_equal(host(y), orc.conv_q(x, w, None, 4, 25, 4, st, pad, g, False)[0])
    # operands at odd addresses, the result in a channel slice of a wider tensor with an odd pitch
    ldy = K + 6
    wide = torch.full((N, y_ref.shape[1], y_ref.shape[2], ldy), 77, dtype=torch.int8, device="cuda")
    B.conv_q(_odd(x, 3), _odd(w, 5), bd, 4, shift, 4, st, pad, g, True, out=wide.view(-1)[1:], ldy=ldy, variant=B.CONV_RAGGED)
    got = host(wide).reshape(-1, ldy)
    assert np.array_equal(got[:, 1:1 + K], y_ref.reshape(-1, K))
    assert (got[:, 0] == 77).all() and (got[:, 1 + K:] == 77).all()
    # one weight format per output channel: inside the range of the packed rounding, from 0 on, and outside it
    for lo, hi in ((-4, shift + 2), (shift - 1, 24)):
        f_w = rng.integers(lo, hi, K).astype(np.int32)
        f_w[:2] = lo, hi - 1
        for relu in (False, True):
            y, _ = B.conv_q_pc(xd, wd, bd, 4, dev(f_w), 0, st, pad, g, relu)
            assert np.array_equal(host(y), orc.conv_q(x, w, b, 4, f_w, 0, st, pad, g, relu)[0])
