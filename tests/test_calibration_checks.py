"""What calibration refuses before a kernel sees it: weights and biases that do not fit the graph, operands that do not fit each other, inputs that
are no codes.  A library that only records its calls stands in for the kernels, host tensors for the device's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl
from paper_1805_07941_amd import binding as B
from paper_1805_07941_amd import net as int8net
from paper_1805_07941_amd import npnet


class Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append(name)
            return B.OK
        return call


@pytest.fixture
def library(monkeypatch):
    rec = Recorder()

    def dev(t, dtype, name):
        if t.dtype != dtype or not t.is_contiguous():
            raise TypeError(name)
        return t
    monkeypatch.setattr(B, "lib", lambda: rec)
    monkeypatch.setattr(B, "status_string", str)
    monkeypatch.setattr(B, "_dev", dev)
    monkeypatch.setattr(B, "_stream", lambda s: None)
    return rec


def _net(int8=False, change=None, channels=8):
    """Two convolutions meet in an add and in a concat; `change`: {layer: (weights, bias) -> (weights, bias)}."""
    net = wl.Net(3, "join", 2, (6, 6, channels))
    net.shapes["input"] = net.in_shape
    net.input_is_int8, net.f_input_codes = int8, 4
    a = net.conv("a", "input", 8, 3, pad=1)
    b = net.conv("b", a, 8, 1)
    net.output_name = net.eltwise("add", a, b)
    plain = net.weights
    net.weights = lambda nd: (change or {}).get(nd.name, lambda *wb: wb)(*plain(nd))
    return net


def _int8(net, x, **kw):
    return int8net.calibrate(net, x, device="cpu", **kw)


def _x(net):
    return torch.zeros((2,) + net.in_shape, dtype=torch.int8 if net.input_is_int8 else torch.float32)


def test_consistent_networks_pass(library):
    for int8 in (False, True):
        net = _net(int8)
        _int8(net, _x(net))
        _int8(net, _x(net), per_channel=True)
    assert {"dfq_cal_weights", "dfq_cal_rescale", "dfq_cal_add"} <= set(library.calls)


@pytest.mark.parametrize("layer", ["a", "b"])
def test_short_bias(library, layer):
    net = _net(change={layer: lambda w, b: (w, b[:-1])})
    for per_channel in (False, True):
        with pytest.raises(B.DfqError) as e:
            _int8(net, _x(net), per_channel=per_channel)
        assert e.value.status == B.ESHAPE
    assert not any("weights" in c for c in library.calls)


@pytest.mark.parametrize("change", [lambda w, b: (np.concatenate([w] * 40), np.concatenate([b] * 40)), lambda w, b: (w, np.concatenate([b, b])),
                                    lambda w, b: (w, b[:, None])])
def test_shapes_the_graph_does_not_say(library, change):
    """More filters than the graph counts, a longer bias, one of another rank: not by the calls whose words the graph counts."""
    net = _net(change={"b": change})
    try:
        _int8(net, _x(net))
    except B.DfqError as e:                              # 320 channels do not add to 8
        assert e.status == B.ESHAPE and net.weights(net.nodes[1])[0].shape[0] == 320
    assert library.calls.count("dfq_cal_weights") == 1 and "dfq_quantize_i32" in library.calls[library.calls.index("dfq_cal_weights"):]


def test_input_channels(library):
    net = _net(change={"a": lambda w, b: (np.ascontiguousarray(w[..., :5]), b)})
    with pytest.raises(B.DfqError) as e:
        _int8(net, _x(net))
    assert e.value.status == B.ESHAPE and "dfq_conv_q_variant" not in library.calls


def test_operands_of_a_join(library):
    net = _net()
    net.nodes[1].stride = 2
    with pytest.raises(B.DfqError) as e:
        _int8(net, _x(net))
    assert e.value.status == B.ESHAPE and "dfq_cal_add" not in library.calls
    net.nodes[2].op = "concat"
    with pytest.raises(B.DfqError) as e:
        _int8(net, _x(net))
    assert e.value.status == B.ESHAPE and "dfq_cal_concat" not in library.calls


def test_codes_as_the_input(library):
    """An input that an add or a concat reads first."""
    for op in ("eltwise", "concat"):
        net = wl.Net(3, "first", 2, (6, 6, 8))
        net.shapes["input"] = net.in_shape
        net.input_is_int8, net.f_input_codes = True, 4
        net.output_name = net.eltwise("j", "input", "input") if op == "eltwise" else net.concat("j", ["input", "input"])
        good = _x(net)
        for bad in (good.float(), good.to(torch.uint8), good.transpose(1, 2)[..., ::2]):
            with pytest.raises(TypeError):
                _int8(net, bad)
        for f in (33, -33, 100):
            net.f_input_codes = f
            with pytest.raises(B.DfqError) as e:
                _int8(net, good)
            assert e.value.status == B.EFMT
        assert not library.calls
        net.f_input_codes = -32
        _int8(net, good)
        library.calls.clear()


def _np(net):
    return npnet.calibrate(net, _x(net), device="cpu")


def test_np_consistent_network_passes(library):
    _np(_net())
    assert {"dfq_cal_np_weights", "dfq_cal_conv_np", "dfq_cal_add_np"} <= set(library.calls)


@pytest.mark.parametrize("layer", ["a", "b"])
def test_np_short_bias(library, layer):
    with pytest.raises(B.DfqError) as e:
        _np(_net(change={layer: lambda w, b: (w, b[:-1])}))
    assert e.value.status == B.ESHAPE and "dfq_cal_np_weights" not in library.calls


def test_np_input_channels(library):
    with pytest.raises(ValueError):
        _np(_net(change={"a": lambda w, b: (np.ascontiguousarray(w[..., :5]), b)}))
    assert "dfq_cal_conv_np" not in library.calls


def test_np_operands_of_a_join(library):
    net = _net()
    net.nodes[1].stride = 2
    with pytest.raises(ValueError):
        _np(net)
    assert "dfq_cal_conv_np" in library.calls and "dfq_cal_add_np" not in library.calls


def test_np_more_filters_than_the_graph_says(library, monkeypatch):
    """The scratch of a layer's thresholds holds one for each of its filters."""
    sizes = {}
    empty = torch.empty

    def record(*args, **kw):
        t = empty(*args, **kw)
        sizes[t.data_ptr()] = t.numel()
        return t

    def weights(w, bias, rows, row_len, p, gamma, *rest):
        library.calls.append("dfq_cal_np_weights")
        assert sizes[gamma] >= rows
        return B.OK
    monkeypatch.setattr(torch, "empty", record)
    library.dfq_cal_np_weights = weights
    net = _net(change={"b": lambda w, b: (np.concatenate([w] * 40), np.concatenate([b] * 40))})
    with pytest.raises(ValueError):                      # the add: 8 and 320 channels
        _np(net)
    assert library.calls.count("dfq_cal_np_weights") == 2


def test_np_results_apart_from_the_operands():
    """Every result of the (8, p) calls where it meets an operand or another result: refused before anything is launched."""
    L = B.lib()
    M = 1 << 20
    # addresses in order of the arguments, with the bytes behind them: 4 rows of 8 values, 32 values
    weights = [M, 2 * M, 4, 8, 4, 3 * M, 4 * M, 5 * M, 6 * M, 7 * M, 8 * M, 9 * M, 10 * M, None]
    for out, other, distance in ((5 + 2, 0, 127), (8, 0, 64), (9, 0, 1), (7, 8, 31), (8, 9, -31), (9, 7, 5), (11, 1, 15), (11, 7, 31), (7, 1, 3), (11, 0, 127)):
        args = list(weights)
        args[out] = args[other] + distance
        assert L.dfq_cal_np_weights(*args) == B.EINVAL, (out, other)
    quantize = [M, 32, 4, 2 * M, 3 * M, 4 * M, 5 * M, 6 * M, None]
    for out, other, distance in ((4, 0, 127), (5, 0, 0), (5, 4, 31)):
        args = list(quantize)
        args[out] = args[other] + distance
        assert L.dfq_cal_np_quantize(*args) == B.EINVAL, (out, other)
    add = [M, 2 * M, 3 * M, 4 * M, 5 * M, 6 * M, 32, 4, 0, 7 * M, 8 * M, 9 * M, 10 * M, 11 * M, None]
    for out, other, distance in ((10, 0, 31), (10, 1, 0), (10, 3, -31), (10, 4, 8), (11, 0, 0), (11, 4, 1), (11, 10, 31)):
        args = list(add)
        args[out] = args[other] + distance
        assert L.dfq_cal_add_np(*args) == B.EINVAL, (out, other)


@pytest.mark.gpu
@pytest.mark.parametrize("per_channel", [False, True])
def test_a_longer_bias_gives_what_its_first_values_give(per_channel):
    rng = np.random.default_rng(3)
    x = torch.from_numpy(rng.standard_normal((2, 6, 6, 8)).astype(np.float32)).cuda()
    longer = lambda w, b: (w, np.concatenate([b, b * 9]))
    want, tw = int8net.calibrate(_net(), x, per_channel=per_channel)
    got, tg = int8net.calibrate(_net(change={"b": longer}), x, per_channel=per_channel)
    assert want.frac == got.frac and all(np.array_equal(want.w_frac[k], got.w_frac[k]) for k in want.w_frac)
    for name, b in want.b.items():
        assert torch.equal(b, got.b[name][:len(b)]) and torch.equal(want.w[name], got.w[name])
    assert all(torch.equal(tw[k], tg[k]) for k in tw)
    if not per_channel:
        want, tw = npnet.calibrate(_net(), x)
        got, tg = npnet.calibrate(_net(change={"b": longer}), x)
        assert want.frac == got.frac and all(torch.equal(u, v) for k in tw for u, v in zip(tw[k], tg[k]))
