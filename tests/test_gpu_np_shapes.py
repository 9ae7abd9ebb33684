"""The forms of the (8, p) matrix-core convolution - split reduction, steps of 64 and of 128 bytes - against the one-output-per-lane kernel, at
the edges of their tiles and steps: plain, with the add, and the calibration's maximum, with formats given and on the device."""
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_dispatch import launched
from test_gpu_npconv import B, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

SHAPES = [
    # N  H   W   C    K   R  S  st pad
    (1, 7, 7, 512, 512, 3, 3, 1, 1),             # 16 x 16
    (1, 5, 5, 64, 16, 3, 3, 2, 1),               # 16 x 16, taps that a step straddles, odd half step
    (1, 1, 1, 2048, 208, 1, 1, 1, 0),
    (1, 3, 5, 192, 48, 1, 1, 1, 0),              # a step and a half
    (8, 7, 7, 512, 512, 3, 3, 1, 1),             # 32 x 32, eight wavefronts
    (3, 13, 11, 128, 80, 3, 3, 1, 2),            # ragged pixel and channel tiles
    (5, 14, 14, 256, 256, 3, 3, 1, 1),           # 32 x 32, four
    (2, 28, 27, 64, 96, 5, 3, 1, 1),
    (2, 14, 14, 1024, 256, 1, 1, 1, 0),          # 32 x 32, eight, unpadded 1x1
    (5, 14, 14, 512, 512, 1, 1, 1, 0),           # ... four
    (5, 14, 14, 192, 384, 3, 3, 1, 1),           # ... four, taps that a step straddles
    (9, 14, 15, 128, 512, 1, 1, 1, 0),           # one step
    (18, 28, 28, 128, 128, 3, 3, 1, 1),          # ring of three
    (27, 14, 14, 1024, 256, 1, 1, 1, 0),
    (19, 29, 28, 256, 96, 3, 3, 2, 1),
    (33, 29, 31, 128, 112, 3, 3, 1, 1),          # one stage, three workgroups per unit
    (45, 30, 30, 256, 64, 1, 1, 1, 0),
    (21, 30, 31, 192, 80, 3, 3, 1, 1),           # steps of 64 bytes
    (40, 9, 9, 128, 272, 17, 1, 1, 8),           # more kernel rows than the masks of 128-byte steps hold
]


def test_every_form_of_the_split_reduction_is_reached(B):
    seen = set()
    calls = []
    for N, H, W, C, K, R, S, st, pad in SHAPES:
        x, w = (torch.zeros(s, dtype=torch.int8, device="cuda") for s in ((N, H, W, C), (K, R, S, C)))
        calls.append(lambda x=x, w=w, a=(st, pad): B.conv_np(x, x, w, w, None, 8, 8, 8, 4, *a, variant=B.CONV_MFMA))
    for name in launched(calls):
        seen.update(re.findall(r"conv_np_sk_kernel<(\d, \d, \d, \d, \d)>", name))
        seen.update(re.findall(r"conv_np_mfma_kernel<128, 64, (\d, \d), false, false, (?:64|128)>", name))
    assert seen == {"1, 1, 8, 2, 0", "1, 1, 8, 2, 1", "1, 1, 8, 2, 2", "2, 2, 8, 1, 0", "2, 2, 8, 1, 1", "2, 2, 8, 1, 2", "2, 2, 4, 1, 0", "2, 2, 4, 1, 1",
                    "2, 2, 4, 1, 2", "3, 2", "3, 1", "1, 3"}


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forms(B, shape):
    N, H, W, C, K, R, S, st, pad = shape
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    draw = lambda lo, hi, s: torch.randint(lo, hi, s, generator=g, device="cuda")
    sign = lambda s: draw(0, 2, s) * 2 - 1

    def planes(s):
        sg = sign(s)
        return (draw(0, 32, s) * sg).to(torch.int8), (draw(0, 64, s) * sg).to(torch.int8)

    x, w = planes((N, H, W, C)), planes((K, R, S, C))
    b = draw(-10 ** 6, 10 ** 6, (K,)).to(torch.int32)
    fw = int(np.log2(np.sqrt(R * S * C) * 1000 * 1000 / 700))
    P, Q = B.conv_out_hw(H, W, R, S, st, pad)
    o = planes((N, P, Q, K))
    for relu, p, f_y in ((True, 4, 8), (False, 5, 6), (True, 7, 8 + fw - 3)):                       # (the last: a shift of 3, the 64-bit conversion)
        want = B.conv_np(*x, *w, b, 8, fw, f_y, p, st, pad, 1, relu, variant=B.CONV_DIRECT)
        got = B.conv_np(*x, *w, b, 8, fw, f_y, p, st, pad, 1, relu, variant=B.CONV_MFMA)
        assert all(torch.equal(u, v) for u, v in zip(got, want))
        if p != 7:
            add = B.conv_np_add(*x, *w, b, *o, 8, fw, f_y, relu, 7, 5, p, not relu, stride=st, pad=pad)
            ref = B.eltwise_np(*want[1:], f_y, *o, 7, 5, p, not relu)
            assert torch.equal(add[0], ref[1]) and torch.equal(add[1], ref[2])
    for relu in (True, False):
        m = B.conv_np_absmax(*x, *w, b, st, pad, 1, relu)
        f = B.np_frac_from_absmax_u64(m, 8 + fw, 8, 4)
        words = torch.tensor([8, fw, 99, 0], dtype=torch.int32, device="cuda")
        amax = torch.zeros(B.CAL_AMAX_WORDS, dtype=torch.int64, device="cuda")
        y = [torch.empty((N, P, Q, K), dtype=torch.int8, device="cuda") for _ in range(2)]
        at = [words.data_ptr() + 4 * i for i in range(4)]
        B._check(B.lib().dfq_cal_conv_np(*(t.data_ptr() for t in (*x, *w, b, *y)), N, H, W, C, K, R, S, st, pad, 1, at[0], at[1], amax.data_ptr(), 0, 0, at[2], 4,
                                         int(relu), at[3], None), "dfq_cal_conv_np")
        assert int(amax.max()) == m
        assert words.tolist() == [8, fw, f, 0]
        want = B.conv_np(*x, *w, b, 8, fw, f, 4, st, pad, 1, relu, variant=B.CONV_DIRECT)
        assert torch.equal(y[0], want[1]) and torch.equal(y[1], want[2])


@pytest.mark.parametrize("n", [1, 100, 40016, 1000003])
def test_add_with_formats_on_the_device(B, n):
    rng = np.random.default_rng(n)
    beta = rng.integers(-1984, 1985, (2, n))
    beta[0, n // 2], beta[1, n // 2] = 1984, 1984
    split = lambda v: (dev((np.sign(v) * (np.abs(v) >> 6)).astype(np.int8)), dev((np.sign(v) * (np.abs(v) & 63)).astype(np.int8)))
    a, b = split(beta[0]), split(beta[1])
    for fa, fb, relu in ((5, 5, 0), (3, 9, 1), (18, 0, 0)):
        words = torch.tensor([fa, fb, 99, 0], dtype=torch.int32, device="cuda")
        at = [words.data_ptr() + 4 * i for i in range(4)]
        amax = torch.zeros(B.CAL_AMAX_WORDS, dtype=torch.int64, device="cuda")
        y = [torch.empty(n, dtype=torch.int8, device="cuda") for _ in range(2)]
        call = lambda: B._check(B.lib().dfq_cal_add_np(a[0].data_ptr(), a[1].data_ptr(), at[0], b[0].data_ptr(), b[1].data_ptr(), at[1], n, 4, relu,
                                                       amax.data_ptr(), y[0].data_ptr(), y[1].data_ptr(), at[2], at[3], None), "dfq_cal_add_np")
        call()
        m = B.eltwise_np_absmax(*a, fa, *b, fb, bool(relu))
        f = B.np_frac_from_absmax_u64(m, max(fa, fb), 8, 4)
        assert int(amax.max()) == m and words.tolist() == [fa, fb, f, 0]
        want = B.eltwise_np(*a, fa, *b, fb, f, 4, bool(relu))
        assert torch.equal(y[0], want[1]) and torch.equal(y[1], want[2])
    words[0], words[1] = 0, 19
    call()
    assert int(words[3]) == 2                         # what eltwise_np refuses
