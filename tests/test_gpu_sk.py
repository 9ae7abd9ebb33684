"""The dense kernel that splits the reduction inside a workgroup (conv_sk.hip) against the oracle: edges of its tiles, steps and
rings in each of its shapes, and the fused add on both sides of the line behind which the other kernels take it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W    C    K   R  S  st pad
    (1, 1, 1, 16, 1, 1, 1, 1, 0),                # one output, an eighth of a step
    (1, 4, 4, 128, 16, 1, 1, 1, 0),              # exactly one 16 x 16 tile and one step
    (1, 17, 1, 1024, 17, 1, 1, 1, 0),            # tile + 1 both ways, one step per wavefront
    (1, 5, 3, 1152, 33, 1, 1, 1, 0),             # one wavefront has a second step
    (1, 1, 1, 2048, 1000, 1, 1, 1, 0),           # fully connected, the ring wraps
    (3, 7, 5, 4224, 30, 1, 1, 1, 0),             # 33 steps: five on one wavefront, four on the others
    (2, 9, 7, 64, 70, 3, 3, 1, 1),               # a step holds two taps
    (2, 9, 7, 128, 48, 3, 3, 2, 1),              # a tap per step
    (1, 8, 6, 48, 20, 5, 3, 1, 2),               # steps that straddle taps, tail of a step, padding
    (1, 3, 3, 80, 19, 3, 3, 1, 3),               # outputs wholly in the padding
    (1, 40, 6, 16, 10, 31, 3, 1, 15),
    (1, 31, 33, 128, 544, 1, 1, 1, 0),           # 32 x 32 tiles, four wavefronts, one step
    (2, 14, 14, 640, 544, 1, 1, 1, 0),           # 32 x 32 tiles, eight wavefronts, five steps
    (4, 14, 14, 256, 255, 3, 3, 1, 1),           # 18 steps over eight wavefronts, ragged channel tail
    (12, 7, 7, 512, 512, 3, 3, 1, 1),            # 36 steps over four
    (9, 23, 23, 48, 96, 3, 3, 1, 1),
    (4, 28, 28, 128, 128, 3, 3, 2, 1),
    (40, 15, 15, 48, 68, 1, 1, 1, 0),            # by name only: another kernel is faster
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_conv_split_reduction(B, shape):
    N, H, W, C, K, R, S, st, pad = shape
    rng = np.random.default_rng(sum(shape))
    x, w = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (K, R, S, C)).astype(np.int8)
    b = rng.integers(-2 ** 15, 2 ** 15, (K,)).astype(np.int32)
    xd, wd, bd = dev(x), dev(w), dev(b)
    shift = max(0, int(np.log2(np.sqrt(R * S * C) * 70 * 70 / 40)))
    for i, (relu, bias, s) in enumerate([(True, True, shift), (False, False, shift - 2), (True, True, 24), (False, True, -9)]):
        y_ref, acc_ref = orc.conv_q(x, w, b if bias else None, 4, s, 4, st, pad, 1, relu, want_acc=True)
        y, acc = B.conv_q(xd, wd, bd if bias else None, 4, s, 4, st, pad, 1, relu, want_acc=i == 0, variant=B.CONV_SPLIT)
        assert np.array_equal(host(y), y_ref), (relu, bias, s)
        if i == 0:
            assert np.array_equal(host(acc), acc_ref)
            _, acc = B.conv_q(xd, wd, bd, 4, s, 4, st, pad, 1, relu, want_y=False, want_acc=True, variant=B.CONV_SPLIT)
            assert np.array_equal(host(acc), acc_ref)
    # a channel slice of a wider tensor: at a word boundary, and at an odd address and pitch
    y_ref, _ = orc.conv_q(x, w, b, 4, shift, 4, st, pad, 1, True)
    for ldy, off in ((4 * (K // 4) + 8, 4), (K + 7 + K % 2, 1)):
        wide = torch.full((N, y_ref.shape[1], y_ref.shape[2], ldy), 77, dtype=torch.int8, device="cuda")
        B.conv_q(xd, wd, bd, 4, shift, 4, st, pad, 1, True, out=wide.view(-1)[off:], ldy=ldy, variant=B.CONV_SPLIT)
        got = host(wide).reshape(-1, ldy)
        assert np.array_equal(got[:, off:off + K], y_ref.reshape(-1, K))
        assert (got[:, :off] == 77).all() and (got[:, off + K:] == 77).all()
    # one weight format per output channel
    f_w = rng.integers(max(0, shift - 3), shift + 2, K).astype(np.int32)
    y_ref, _ = orc.conv_q(x, w, b, 4, f_w, 4, st, pad, 1, False)
    y, _ = B.conv_q_pc(xd, wd, bd, 4, dev(f_w), 4, st, pad, 1, False)
    assert np.array_equal(host(y), y_ref)


@pytest.mark.parametrize("shape", [(1, 7, 7, 512, 2048), (1, 14, 14, 256, 768), (1, 14, 14, 640, 768),                # split reduction, its three shapes
                                   (23, 27, 31, 64, 256), (19, 21, 19, 192, 320), (9, 37, 41, 256, 384),             # input-resident
                                   (1, 14, 14, 256, 1024), (6, 28, 28, 128, 512), (31, 14, 14, 256, 1024),           # dense: 64 x 64, 128 x 128
                                   (13, 31, 31, 128, 768), (19, 21, 19, 320, 256)],                                  # dense: 128 x 64, steps of 64 bytes
                         ids=lambda s: "x".join(map(str, s)))
def test_fused_add_by_size(B, shape):
    N, H, W, C, K = shape
    rng = np.random.default_rng(sum(shape))
    x, w = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (K, 1, 1, C)).astype(np.int8)
    b, other = rng.integers(-2 ** 15, 2 ** 15, (K,)).astype(np.int32), rng.integers(-128, 128, (N, H, W, K)).astype(np.int8)
    xd, wd, bd, od = dev(x), dev(w), dev(b), dev(other)
    for f_in, f_w, f_mid, relu_mid, f_other, f_out, relu_out in [(4, 8, 4, False, 5, 3, True), (3, 7, 2, True, 1, 0, False), (4, 8, 4, False, 4, 4, True)]:
        mid, _ = orc.conv_q(x, w, b, f_in, f_w, f_mid, 1, 0, 1, relu_mid)
        ref, _ = orc.eltwise_q(mid, f_mid, other, f_other, f_out, relu_out)
        got = B.conv_q_add(xd, wd, bd, od, f_in, f_w, f_mid, relu_mid, f_other, f_out, relu_out)
        assert got is not None and np.array_equal(host(got), ref)
        got = B.conv_q_add_lazy(xd, wd, bd, od, f_in, f_w, f_other, f_out, relu_out)
        ref = orc.conv_q_add_lazy(x, w, b, other, f_in, f_w, f_other, f_out, relu=relu_out)
        assert got is not None and np.array_equal(host(got), ref)
        f_wk = rng.integers(f_w - 2, f_w + 2, K).astype(np.int32)
        mid, _ = orc.conv_q(x, w, b, f_in, f_wk, f_mid, 1, 0, 1, relu_mid)
        ref, _ = orc.eltwise_q(mid, f_mid, other, f_other, f_out, relu_out)
        got = B.conv_q_pc_add(xd, wd, bd, od, f_in, dev(f_wk), (f_w - 2, f_w + 1), f_mid, relu_mid, f_other, f_out, relu_out)
        # per-channel formats over at most 1024 pixels are declined where the input-resident kernel's buffers and tables do not fit
        if N * H * W <= 1024 and (C > 256 or 512 * C + 192 * (64 if K % 128 else 128) + 16 * K > 160 * 1024):
            assert got is None
        else:
            assert got is not None and np.array_equal(host(got), ref)


@pytest.mark.parametrize("shape", [(1, 64, 64, 3, 64, 7, 7, 2, 3), (3, 36, 64, 3, 32, 3, 3, 2, 1), (2, 44, 96, 3, 64, 3, 3, 2, 0), (1, 33, 37, 3, 50, 7, 7, 2, 3),
                                   (2, 20, 31, 1, 7, 5, 5, 1, 2), (1, 40, 33, 2, 100, 3, 16, 1, 1), (1, 12, 33, 3, 3, 1, 1, 1, 0)], ids=lambda s: "x".join(map(str, s)))
def test_first_layer_weights(B, shape):
    """First layers: weight runs of every length, the last run of the tensor, strips of one step, channels with shifts inside and
    outside the lean range."""
    N, H, W, C, K, R, S, st, pad = shape
    rng = np.random.default_rng(sum(shape))
    x, w = rng.integers(-128, 128, (N, H, W, C)).astype(np.int8), rng.integers(-128, 128, (K, R, S, C)).astype(np.int8)
    b = rng.integers(-2 ** 12, 2 ** 12, (K,)).astype(np.int32)
    wd = dev(w)
    for relu in (False, True):
        y_ref, _ = orc.conv_q(x, w, b, 4, 8, 4, st, pad, 1, relu)
        assert np.array_equal(host(B.conv_q(dev(x), wd, dev(b), 4, 8, 4, st, pad, 1, relu)[0]), y_ref)
        for lo, hi in ((5, 10), (-3, 28)):
            f_w = rng.integers(lo, hi + 1, K).astype(np.int32)
            y_ref, _ = orc.conv_q(x, w, b, 4, f_w, 4, st, pad, 1, relu)
            assert np.array_equal(host(B.conv_q_pc(dev(x), wd, dev(b), 4, dev(f_w), 4, st, pad, 1, relu, frac_w_range=(lo, hi))[0]), y_ref)
