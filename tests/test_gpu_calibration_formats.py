"""Formats chosen on the device against the host rules: thresholds at the edges of every format, alignment limits, infinities."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as orc

from test_gpu_ops import B, dev, host            # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


class Words:
    def __init__(self, *values):
        self.t = torch.tensor(list(values) + [0, 0, 0, 0], dtype=torch.int32, device="cuda")
        self.n = len(values)

    def at(self, i):
        return self.t.data_ptr() + 4 * i


@pytest.mark.parametrize("row_len", [1, 3, 36, 1000])
@pytest.mark.parametrize("per_row", [0, 1])
def test_weights(B, row_len, per_row):
    rng = np.random.default_rng(row_len + per_row)
    rows = 37
    w = (rng.standard_normal((rows, row_len)) * 2.0 ** rng.integers(-30, 30, (rows, 1))).astype(np.float32)
    for r, top in enumerate([0.0, 127.0, np.nextafter(np.float32(127.0), np.float32(1e9)), 128.0, 1.0, 2.0 ** -140, 3e38, 127.0 * 2.0 ** -32, 2.0 ** 39]):
        w[r] = 0.0
        w[r, row_len // 2] = -top                      # NaN is skipped
        if row_len > 1:
            w[r, 0 if row_len // 2 else 1] = np.nan
    bias = (rng.standard_normal(rows) * 1000).astype(np.float32)
    f_in = 5
    W = Words(f_in)
    wd, bd = dev(w), dev(bias)
    q, b = torch.empty((rows, row_len), dtype=torch.int8, device="cuda"), torch.empty(rows, dtype=torch.int32, device="cuda")
    w_frac, gamma = torch.full((rows,), 99, dtype=torch.int32, device="cuda"), torch.empty(rows, device="cuda")
    B._check(B.lib().dfq_cal_weights(wd.data_ptr(), bd.data_ptr(), rows, row_len, per_row, gamma.data_ptr(), W.at(0), q.data_ptr(), w_frac.data_ptr(),
                                     b.data_ptr(), W.at(1), None), "dfq_cal_weights")
    top = np.nan_to_num(np.abs(w)).max(axis=1) if per_row else np.full(1, np.nan_to_num(np.abs(w)).max())
    want = np.array([B.fmt_from_absmax_f32(float(g)) for g in top], dtype=np.int32)
    assert np.array_equal(host(w_frac)[:len(want)], want) and host(W.t)[1] == 0
    frac = want if per_row else np.repeat(want, rows)
    assert np.array_equal(host(q), host(B.quantize_rows(wd, dev(frac))))
    assert np.array_equal(host(b), host(B.quantize_i32_rows(bd, dev(frac), f_in)))
    w[5] = np.inf
    wd = dev(w)
    B._check(B.lib().dfq_cal_weights(wd.data_ptr(), bd.data_ptr(), rows, row_len, per_row, gamma.data_ptr(), W.at(0), q.data_ptr(), w_frac.data_ptr(),
                                     b.data_ptr(), W.at(1), None), "dfq_cal_weights")
    assert host(W.t)[1] == 1


@pytest.mark.parametrize("K", [1, 3, 8, 300])
@pytest.mark.parametrize("per_channel", [0, 1])
def test_rescale(B, K, per_channel):
    rng = np.random.default_rng(K + per_channel)
    for pixels, top in ((1, 127), (1, 128), (3, 0), (700, 254), (700, 255), (5000, 2 ** 31 - 1)):
        acc = rng.integers(-max(top, 1), max(top, 1), (pixels, K)).astype(np.int32) if top else np.zeros((pixels, K), np.int32)
        acc[pixels // 2, K // 2] = top
        for f_in, relu, fixed in ((4, 0, None), (-20, 1, None), (32, 1, None), (3, 0, 1)):
            f_w = rng.integers(-3, 12, K if per_channel else 1).astype(np.int32)
            W = Words(f_in)
            y = torch.empty((pixels, K), dtype=torch.int8, device="cuda")
            maxima = torch.zeros(K, dtype=torch.int32, device="cuda")
            ad, fd = dev(acc), dev(f_w)
            B._check(B.lib().dfq_cal_rescale(ad.data_ptr(), pixels, K, relu, W.at(0), fd.data_ptr(), per_channel, maxima.data_ptr(), int(fixed is not None),
                                             fixed or 0, y.data_ptr(), W.at(1), None), "dfq_cal_rescale")
            if fixed is not None:
                f = fixed
            else:
                m = (np.maximum(acc.astype(np.int64), 0) if relu else np.abs(acc.astype(np.int64))).max(axis=0)
                fw = np.broadcast_to(f_w, K)
                f = min(B.fmt_from_absmax_i32(int(m[k]), f_in + int(fw[k])) for k in range(K))
            assert host(W.t)[1] == f
            # the convolution's own rescale of the same sums: a 1x1 layer whose products are zero, every sum the bias of a channel of its own
            want = orc.conv_q(np.zeros((1, 1, 1, 1), np.int8), np.zeros((pixels * K, 1, 1, 1), np.int8), acc.reshape(-1), f_in,
                              np.tile(f_w, pixels) if per_channel else int(f_w[0]), f, 1, 0, 1, bool(relu))[0].reshape(pixels, K)
            assert np.array_equal(host(y), want)


@pytest.mark.parametrize("n", [1, 4, 1001, 40000])
def test_add(B, n):
    rng = np.random.default_rng(n)
    a, b = (rng.integers(-128, 128, n).astype(np.int8) for _ in range(2))
    ad, bd = dev(a), dev(b)
    for fa, fb, relu in ((4, 4, 0), (7, 2, 1), (-3, 19, 0), (0, 22, 1)):
        W = Words(fa, fb)
        y, mx = torch.empty(n, dtype=torch.int8, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        call = lambda: B._check(B.lib().dfq_cal_add(ad.data_ptr(), W.at(0), bd.data_ptr(), W.at(1), n, relu, mx.data_ptr(), y.data_ptr(), W.at(2), W.at(3),
                                                    None), "dfq_cal_add")
        call()
        _, acc = B.eltwise_q(ad, fa, bd, fb, 0, bool(relu), want_y=False, want_acc=True)
        f = B.fmt_from_absmax_i32(B.absmax_i32_value(B.absmax_i32(acc, relu=bool(relu))), max(fa, fb))
        got = host(W.t)
        assert got[2] == f and got[3] == 0
        assert np.array_equal(host(y), host(B.eltwise_q(ad, fa, bd, fb, f, bool(relu))[0]))
    W = Words(0, 23)
    mx.zero_()
    call()
    assert host(W.t)[3] == 2                               # what eltwise_q refuses


def test_concat(B):
    rng = np.random.default_rng(0)
    for Cs, fixed in (((3, 64), None), ((16, 17, 40), None), ((5, 5), 2), ((32, 48), None)):
        xs = [rng.integers(-128, 128, (2, 5, 7, c)).astype(np.int8) for c in Cs]
        fs = [int(v) for v in rng.integers(2, 9, len(Cs))]
        W = Words(*fs)
        xd = [dev(x) for x in xs]
        import ctypes as C
        nb = len(Cs)
        y = torch.empty((2, 5, 7, sum(Cs)), dtype=torch.int8, device="cuda")
        B._check(B.lib().dfq_cal_concat(nb, (C.c_void_p * nb)(*[x.data_ptr() for x in xd]), (C.c_int * nb)(*Cs), W.at(0), (C.c_int * nb)(*range(nb)),
                                        int(fixed is not None), fixed or 0, y.data_ptr(), W.at(nb), 70, None), "dfq_cal_concat")
        f = fixed if fixed is not None else min(fs)
        assert host(W.t)[nb] == f
        assert np.array_equal(host(y), host(B.concat_q(xd, fs, f)))


def test_infinite_threshold_is_refused(B):
    import workloads as wl
    from paper_1805_07941_amd import net as int8net, npnet
    net = wl.resnet50(batch=1, hw=32, classes=10)
    x = torch.randn((1, 32, 32, 3), device="cuda")
    plain = net.weights
    for bad in (np.inf, -np.inf):
        def weights(nd):
            w, b = plain(nd)
            if nd is net.nodes[2]:
                w = w.copy()
                w.flat[3] = bad
            return w, b
        net.weights = weights
        for run in (lambda: int8net.calibrate(net, x), lambda: int8net.calibrate(net, x, per_channel=True), lambda: npnet.calibrate(net, x)):
            with pytest.raises(B.DfqError):
                run()
