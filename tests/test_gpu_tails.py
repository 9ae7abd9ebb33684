"""Channel tails of the dense kernel (whole groups of sixteen past a tile's last full part, single channels), its accumulator dump, and
the pooling kernels that share reads between windows or pixels between lanes: against the oracle at the edges of their tiles."""
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc
import oracle.npconv as NC

from test_gpu_dispatch import launched
from test_gpu_npnet import planes
from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [8, 16, 31, 48, 63, 80, 96, 112, 127, 176, 192])
@pytest.mark.parametrize("geo", [(37, 11, 13, 96, 1, 1), (19, 17, 15, 48, 3, 1), (24, 21, 20, 64, 3, 2), (30, 14, 13, 128, 1, 1), (17, 16, 16, 128, 3, 1)],
                         ids=lambda g: "x".join(map(str, g)))
def test_channel_tails(B, geo, K):
    N, H, W, C, R, st = geo
    rng = np.random.default_rng(K + sum(geo))
    x, w = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (K, R, R, C)).astype(np.int8)
    b = rng.integers(-2 ** 15, 2 ** 15, (K,)).astype(np.int32)
    xd, wd, bd = dev(x), dev(w), dev(b)
    shift, pad = int(np.log2(R * np.sqrt(C) * 70 * 70 / 40)), R // 2
    y_ref, acc_ref = orc.conv_q(x, w, b, 4, shift, 4, st, pad, 1, True, want_acc=True)
    got = B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, 1, True, variant=B.CONV_MFMA)[0]
    assert np.array_equal(host(got), y_ref)
    # sums alone, and beside the codes
    for want_y in (False, True):
        y, acc = B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, 1, True, want_y=want_y, want_acc=True, variant=B.CONV_MFMA)
        assert np.array_equal(host(acc), acc_ref) and (y is None or np.array_equal(host(y), y_ref))
    # into a slice whose pitch keeps rows aligned, and one that does not
    for before, behind in ((16, (-K) % 16 + 16), (3, 4)):
        pitch = before + K + behind
        wide = torch.full((N, y_ref.shape[1], y_ref.shape[2], pitch), 77, dtype=torch.int8, device="cuda")
        B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, 1, True, out=wide.view(-1)[before:], ldy=pitch, variant=B.CONV_MFMA)
        got = host(wide)
        assert np.array_equal(got[..., before:before + K], y_ref)
        assert (got[..., :before] == 77).all() and (got[..., before + K:] == 77).all()
    # one weight format per channel, and a shift beyond the four-instruction rounding
    f_w = rng.integers(shift - 3, shift + 2, K).astype(np.int32)
    assert np.array_equal(host(B.conv_q_pc(xd, wd, bd, 4, dev(f_w), 4, st, pad, 1, False)[0]),
                          orc.conv_q(x, w, b, 4, f_w, 4, st, pad, 1, False)[0])
    assert np.array_equal(host(B.conv_q(xd, wd, bd, 4, 24, 4, st, pad, 1, False, variant=B.CONV_MFMA)[0]),
                          orc.conv_q(x, w, b, 4, 24, 4, st, pad, 1, False)[0])


# Tile shapes (pixels, channels, bytes of a step) that the layers above are too small for.
LARGE = [
    (90, 14, 13, 128, 80, 1, "128, 64, 128"),
    (60, 15, 13, 128, 176, 3, "128, 64, 128"),
    (100, 32, 32, 16, 48, 3, "256, 64, 64"),     # four tiles of 128 pixels to a unit
    (130, 32, 32, 16, 48, 3, "128, 64, 64"),     # five
    (180, 32, 32, 16, 48, 3, "128, 64, 64"),     # six
    (251, 32, 32, 16, 48, 3, "256, 64, 64"),     # eight
    (260, 32, 32, 16, 48, 3, "128, 64, 64"),     # nine
    (420, 32, 32, 16, 48, 3, "256, 64, 64"),     # fourteen
    (400, 31, 32, 16, 48, 1, "256, 64, 64"),
]


@pytest.mark.parametrize("shape", LARGE, ids=lambda s: "x".join(map(str, s[:6])))
def test_channel_tails_of_large_layers(B, shape):
    """Against one output per lane: the shape's last full group of sixteen and none behind it, with the kernel that ran."""
    N, H, W, C, K, R, tile = shape
    g = torch.Generator(device="cuda").manual_seed(K + N)
    x, w = (torch.randint(-128, 128, s, generator=g, device="cuda").to(torch.int8) for s in ((N, H, W, C), (K, R, R, C)))
    b = torch.randint(-2 ** 15, 2 ** 15, (K,), generator=g, device="cuda").to(torch.int32)
    shift = int(np.log2(R * np.sqrt(C) * 70 * 70 / 40))
    want = B.conv_q(x, w, b, 4, shift, 4, 1, R // 2, 1, True, variant=B.CONV_DIRECT)[0]
    wide = torch.full((N, H, W, K + 32), 77, dtype=torch.int8, device="cuda")
    run = lambda: B.conv_q(x, w, b, 4, shift, 4, 1, R // 2, 1, True, out=wide.view(-1)[16:], ldy=K + 32, variant=B.CONV_MFMA)
    run()
    assert torch.equal(wide[..., 16:16 + K], want)
    assert bool((wide[..., :16] == 77).all()) and bool((wide[..., 16 + K:] == 77).all())
    (name,) = launched([run])
    m = re.search(r"conv_mfma_kernel<(\d+), (\d+), .* (\d+)>", name)
    assert ", ".join(m.groups()) == tile


# the first seven in strips of four rows (with a padding at least; the last two of them images of one row and of one column)
POOLS = [(40, 28, 27, 192), (80, 33, 31, 45), (24, 45, 61, 90), (150, 29, 30, 17), (3, 112, 97, 180), (4, 1, 300, 900), (16, 301, 1, 1000),
         (9, 28, 27, 192), (40, 33, 31, 45), (12, 45, 61, 90), (70, 29, 30, 17), (3, 301, 1, 1000)]


def test_strips_are_reached(B):
    calls = [lambda x=torch.zeros(s, dtype=torch.int8, device="cuda"): B.pool_q(x, "max", 3, 1, 1, 4, 4) for s in POOLS]
    calls[0]()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        for call in calls:
            call()
        torch.cuda.synchronize()
    names = [e.name for e in sorted((e for e in prof.events() if "pool" in e.name), key=lambda e: e.time_range.start)]
    if not names:
        pytest.skip("the device's activity is not recorded here")
    assert ["maxpool3_s1_kernel" in name for name in names] == [True] * 7 + [False] * 5


@pytest.mark.parametrize("shape", POOLS, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("pad", [0, 1, 2])
def test_max_pool_strips(B, shape, pad):
    if min(shape[1:3]) + 2 * pad < 3:
        pytest.skip("no window fits")
    rng = np.random.default_rng(sum(shape) + pad)
    x = rng.integers(-128, 128, shape).astype(np.int8)
    x[0] = -128                                       # saturates to -127
    for f_out in (4, 3, 6):
        assert np.array_equal(host(B.pool_q(dev(x), "max", 3, 1, pad, 4, f_out)), orc.pool_q(x, "max", 3, 1, pad, 4, f_out))


@pytest.mark.parametrize("shape", [(1, 7, 2048), (3, 7, 1000), (2, 1, 4), (5, 14, 36), (1, 64, 132), (33, 8, 124), (2, 57, 64)], ids=lambda s: "x".join(map(str, s)))
def test_global_average(B, shape):
    N, k, C = shape
    rng = np.random.default_rng(sum(shape))
    x = rng.integers(-128, 128, (N, k, k, C)).astype(np.int8)
    x[0, ..., :2] = (-128, 127)
    for f_out in (4, 2, 9, 20):
        assert np.array_equal(host(B.pool_q(dev(x), "avg", k, 1, 0, 4, f_out)), orc.pool_q(x, "avg", k, 1, 0, 4, f_out))


@pytest.mark.parametrize("shape", [(1, 7, 2048), (3, 5, 100), (2, 1, 4), (9, 13, 132)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("p", [4, 7])
def test_global_average_of_digit_planes(B, shape, p):
    N, k, C = shape
    rng = np.random.default_rng(sum(shape) + p)
    x = rng.integers(0, 256, (N, k, k, C)).astype(np.uint8)
    ry, rbeta = NC.pool_np(x, (8, p), "avg", k, 1, 0)
    y, yh, yl = B.pool_np(*planes(B, x, p), "avg", k, 1, 0, p)
    assert np.array_equal(host(y), ry)
    assert np.array_equal(64 * host(yh).astype(np.int64) + host(yl), rbeta)


@pytest.mark.parametrize("shape", [(2, 9, 11, 24, 36, 3, 12), (3, 8, 7, 18, 36, 1, 6), (1, 13, 9, 36, 28, 3, 4)], ids=lambda s: "x".join(map(str, s)))
def test_sums_of_groups_that_start_anywhere(B, shape):
    """K is a multiple of four and the outputs of a group are not: a group's sums must not reach into the next one's."""
    N, H, W, C, K, R, g = shape
    rng = np.random.default_rng(sum(shape))
    x, w = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (K, R, R, C // g)).astype(np.int8)
    b = rng.integers(-2 ** 15, 2 ** 15, (K,)).astype(np.int32)
    y_ref, acc_ref = orc.conv_q(x, w, b, 4, 7, 4, 1, R // 2, g, True, want_acc=True)
    y, acc = B.conv_q(dev(x), dev(w), dev(b), 4, 7, 4, 1, R // 2, g, True, want_acc=True, variant=B.CONV_RAGGED)
    assert np.array_equal(host(acc), acc_ref) and np.array_equal(host(y), y_ref)
