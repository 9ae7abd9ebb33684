"""Grouped layers on the matrix cores (conv_sg.hip) against the oracle: every group size and tap count, both widths of a channel block, one tile and
several per workgroup, ragged last tiles."""
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_dispatch import launched
from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W    C   Cg  R  S  st pad
    (1, 1, 1, 64, 4, 1, 1, 1, 0),
    (2, 9, 7, 128, 8, 3, 3, 1, 1),
    (3, 11, 13, 192, 16, 3, 3, 2, 1),            # three blocks of 64 channels
    (2, 10, 9, 256, 32, 2, 3, 1, 1),
    (1, 12, 11, 384, 16, 4, 1, 1, 0),            # three blocks of 128
    (2, 8, 9, 192, 64, 4, 1, 1, 2),
    (41, 59, 57, 64, 8, 3, 3, 1, 1),             # two tiles per workgroup, ragged
    (23, 57, 59, 128, 4, 4, 1, 1, 1),
    (24, 60, 59, 128, 64, 2, 3, 1, 0),
    (50, 60, 45, 64, 32, 1, 1, 1, 0),            # one tap: a tile to a workgroup
    (9, 61, 60, 384, 16, 3, 3, 1, 1),
    (3, 9, 8, 128, 16, 1, 1, 1, 0),              # the other triples of taps, width and group that there are
    (45, 60, 45, 128, 64, 1, 1, 1, 0),
    (4, 7, 9, 192, 64, 1, 1, 1, 0),
    (3, 10, 9, 64, 16, 4, 1, 1, 1),
    (2, 11, 9, 128, 64, 4, 1, 2, 0),
    (3, 9, 10, 64, 16, 2, 3, 1, 1),
]


def test_every_form_is_reached(B):
    calls = []
    for N, H, W, C, Cg, R, S, st, pad in SHAPES:
        x, w = (torch.zeros(s, dtype=torch.int8, device="cuda") for s in ((N, H, W, C), (C, R, S, Cg)))
        calls.append(lambda x=x, w=w, a=(st, pad, C // Cg): B.conv_q(x, w, None, 4, 8, 4, *a, variant=B.CONV_GROUPED))
    seen = {tuple(int(v) for v in m) for name in launched(calls) for m in re.findall(r"conv_sg_kernel<(\d), \d, (\d+), (\d), \d>", name)}
    # (the weights of a grouped layer are at most 64 KB: groups of 64 have six taps in 128 channels, four in 192)
    assert seen == {(taps, width, 1) for taps in (1, 4, 6, 9) for width in (64, 128)} | {(1, 64, 2), (4, 64, 2), (1, 128, 2), (4, 128, 2), (6, 128, 2)}


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_sg(B, shape):
    N, H, W, C, Cg, R, S, st, pad = shape
    rng = np.random.default_rng(sum(shape))
    g = C // Cg
    x, w = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (C, R, S, Cg)).astype(np.int8)
    b = rng.integers(-2 ** 13, 2 ** 13, (C,)).astype(np.int32)
    shift = int(np.log2(np.sqrt(R * S * Cg) * 70 * 70 / 40))
    for relu, bias, s in ((True, b, shift), (False, None, 0)):
        y_ref, _ = orc.conv_q(x, w, bias, 4, s, 4, st, pad, g, relu)
        wide = torch.full((N, y_ref.shape[1], y_ref.shape[2], C + 32), 77, dtype=torch.int8, device="cuda")
        B.conv_q(dev(x), dev(w), None if bias is None else dev(bias), 4, s, 4, st, pad, g, relu, out=wide.view(-1)[16:], ldy=C + 32,
                 variant=B.CONV_GROUPED)
        got = host(wide)
        assert np.array_equal(got[..., 16:16 + C], y_ref)
        assert (got[..., :16] == 77).all() and (got[..., 16 + C:] == 77).all()
