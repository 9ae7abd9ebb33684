"""Ragged layers whose input rows are staged in LDS (conv_rag.hip) against the oracle: tiles that cross images, rows that end inside a piece,
strides up to the kernel's size and beyond, channel tails, operands at odd addresses."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_dispatch import launched
from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)
from test_gpu_ragged import _case, _odd

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W    C    K   R  S  st pad
    (5, 7, 9, 71, 33, 3, 3, 1, 1),              # a tile crosses three images; ten steps and a half
    (19, 3, 12, 73, 31, 3, 3, 1, 1),            # five images in a tile
    (40, 1, 16, 51, 40, 5, 5, 1, 2),            # images of one row
    (2, 33, 41, 83, 131, 3, 3, 1, 1),
    (2, 19, 21, 97, 64, 3, 5, 1, 2),            # wider than high
    (3, 24, 23, 69, 70, 5, 3, 2, 2),
    (2, 31, 131, 39, 65, 3, 15, 3, 7),          # stride = the kernel's height: rows have no slot twice
    (2, 30, 139, 29, 32, 3, 15, 5, 1),          # stride beyond it: rows in between have none
    (3, 9, 60, 67, 40, 1, 9, 1, 4),             # a kernel of one row, images with rows of padding alone
    (1, 12, 70, 45, 20, 5, 5, 1, 4),            # padding as wide as the kernel allows outputs for
    (30, 30, 31, 79, 96, 3, 3, 1, 1),           # more tiles than two per unit: 64 channels each
    (44, 28, 28, 107, 100, 3, 3, 1, 1),
    (1, 15, 16, 33, 7, 35, 3, 1, 17),           # many kernel rows
    (1, 9, 128, 83, 9, 5, 5, 1, 2),             # rows of 10 KB
]
# the same kinds where the rows do not fit, or take too many rounds of loads for their steps
ELSEWHERE = [
    (40, 1, 1, 130, 40, 3, 3, 1, 1),
    (2, 29, 31, 123, 65, 3, 3, 3, 1),
    (2, 30, 31, 117, 32, 3, 3, 5, 1),
    (19, 3, 3, 75, 31, 3, 3, 1, 1),
    (40, 1, 1, 83, 40, 3, 3, 1, 1),
    (2, 31, 131, 39, 65, 3, 9, 3, 1),
    (3, 17, 60, 29, 33, 5, 7, 6, 2),
    (1, 9, 128, 83, 9, 3, 3, 1, 1),
]


def test_kernels_of_the_shapes(B):
    """Which kernel the calls below reach, read from the device's records: these tests are about conv_rag_kernel_rows."""
    calls = []
    for N, H, W, C, K, R, S, st, pad in SHAPES + ELSEWHERE:
        x = torch.randint(-128, 128, (N, H, W, C), dtype=torch.int8, device="cuda")
        w = torch.randint(-128, 128, (K, R, S, C), dtype=torch.int8, device="cuda")
        f = torch.full((K,), 8, dtype=torch.int32, device="cuda")
        calls += [lambda x=x, w=w, a=(st, pad, 1): B.conv_q(x, w, None, 4, 8, 4, *a, True, variant=B.CONV_RAGGED),
                  lambda x=x, w=w, a=(st, pad, 1): B.conv_q(x, w, None, 4, 8, 4, *a, True, want_acc=True, variant=B.CONV_RAGGED),
                  lambda x=x, w=w, f=f, a=(st, pad, 1): B.conv_q_pc(x, w, None, 4, f, 4, *a, True, frac_w_range=(8, 8))]
    got = launched(calls)
    assert len(got) == len(calls)
    assert ["conv_rag_kernel_rows" in name for name in got] == [True] * (3 * len(SHAPES)) + [False] * (3 * len(ELSEWHERE))


@pytest.mark.parametrize("shape", SHAPES + ELSEWHERE, ids=lambda s: "x".join(map(str, s)))
def test_rows(B, shape):
    N, H, W, C, K, R, S, st, pad = shape
    rng = np.random.default_rng(sum(shape))
    x, w, b = _case(rng, shape + (1,))
    shift = max(0, int(np.log2(np.sqrt(R * S * C) * 70 * 70 / 40)))
    y_ref, acc_ref = orc.conv_q(x, w, b, 4, shift, 4, st, pad, 1, True, want_acc=True)
    y, acc = B.conv_q(dev(x), dev(w), dev(b), 4, shift, 4, st, pad, 1, True, want_acc=True, variant=B.CONV_RAGGED)
    assert np.array_equal(host(acc), acc_ref) and np.array_equal(host(y), y_ref)
    for off in (1, 2, 3):
        wide = torch.full((N, y_ref.shape[1], y_ref.shape[2], K + 5), 77, dtype=torch.int8, device="cuda")
        B.conv_q(_odd(x, off), _odd(w, 4 - off), dev(b), 4, shift, 4, st, pad, 1, True, out=wide.view(-1)[off:], ldy=K + 5, variant=B.CONV_RAGGED)
        got = host(wide).reshape(-1)
        pixels = y_ref.size // K
        rows = np.lib.stride_tricks.as_strided(got[off:], (pixels, K), (K + 5, 1))
        assert np.array_equal(rows, y_ref.reshape(pixels, K))
        keep = np.ones(got.size, bool)
        for i in range(pixels):
            keep[off + i * (K + 5):off + i * (K + 5) + K] = False
        assert (got[keep] == 77).all()
    f_w = rng.integers(max(0, shift - 3), shift + 2, K).astype(np.int32)
    y_ref, _ = orc.conv_q(x, w, None, 4, f_w, 4, st, pad, 1, False)
    assert np.array_equal(host(B.conv_q_pc(dev(x), dev(w), None, 4, dev(f_w), 4, st, pad, 1, False)[0]), y_ref)
