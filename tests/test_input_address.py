"""A plan's calls on inputs at other addresses: built once for a shape, the input's address replaced wherever it stands."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl
from paper_1805_07941_amd import binding as B
from paper_1805_07941_amd import net as int8net


def _flat(calls):
    """Arguments of a list of calls with the contents of arrays in place of the arrays."""
    return [(fn.__name__, [list(a) if isinstance(a, C.Array) and a._type_ is C.c_void_p else
                           [v.frac for v in a] if isinstance(a, C.Array) and a._type_ is B.Fmt else
                           list(a) if isinstance(a, C.Array) else a.frac if isinstance(a, B.Fmt) else a for a in args]) for fn, args in calls]


def _records(calls):
    """The words of the records, those that hold an array's address blanked (and what the array holds beside them)."""
    words = list(B.CallList(calls)._records) if not isinstance(calls, B.CallList) else list(calls._records)
    held = calls if not isinstance(calls, B.CallList) else calls._held
    for i, (fn, args) in enumerate(held):
        for j, a in enumerate(args):
            if isinstance(a, C.Array):
                at = i * (B.CALL_ARGS + 1) + 1 + j
                assert words[at] == C.addressof(a)
                words[at] = -1
    return words


def _joined(int8):
    """The input in a convolution, a pooling, an add with itself and at both ends of a concat."""
    net = wl.Net(3, "uses", 2, (6, 6, 16), input_is_int8=int8)
    net.shapes["input"] = net.in_shape
    net.f_input_codes = 4
    a = net.conv("a", "input", 16, 3, pad=1)
    p = net.pool("maxpool", "p", "input", 3, 1, pad=1)
    e = net.eltwise("e", "input", "input")
    net.output_name = net.concat("c", ["input", a, p, e, "input"])
    return net


def _host_plan(net):
    qz = int8net.Quantized()
    qz.frac = {name: 4 for name in [net.input_name] + [nd.dst for nd in net.nodes]}
    for nd in net.nodes:
        if nd.op == "conv":
            qz.w_frac[nd.name] = 5
            qz.w[nd.name] = torch.zeros((nd.K, nd.R, nd.R, net.shapes[nd.srcs[0]][2]), dtype=torch.int8)
            qz.b[nd.name] = torch.zeros(nd.K, dtype=torch.int32)
    return int8net.Plan(net, qz, net.batch, device="cpu")


@pytest.mark.parametrize("int8", [False, True])
def test_calls_are_built_once_for_a_shape(int8, monkeypatch):
    net = _joined(int8)
    plan = _host_plan(net)
    builds = []
    build = int8net.Plan._build_calls
    monkeypatch.setattr(int8net.Plan, "_build_calls", lambda self, x: builds.append(tuple(x.shape)) or build(self, x))
    store = torch.zeros(1 << 16, dtype=torch.int8 if int8 else torch.float32)
    start = (-store.data_ptr() % 256) // store.element_size()
    size = int(np.prod((2,) + net.in_shape))
    step = (size * store.element_size() + 255) // 256 * 256 // store.element_size()
    xs = [store[start + i * step:start + i * step + size].view((2,) + net.in_shape) for i in range(3)]
    seen = []
    for x in (xs[0], xs[1], xs[1], xs[0], xs[2]):
        calls = plan._calls_for(x)
        assert calls is plan._calls and plan._graph is None
        want = build(plan, x)
        assert _flat(calls) == _flat(want)
        assert _records(plan._list) == _records(want)
        if int8:
            assert plan.buf[net.input_name].data_ptr() == x.data_ptr()
        seen.append((calls, _flat(calls)))
    assert len(builds) == 1
    for calls, flat in seen:                                 # a list handed out before stays what it was
        assert _flat(calls) == flat
    # another shape, and an address of other alignment: built anew
    plan._calls_for(xs[0][:1])
    plan._calls_for(xs[0])
    odd = store[start + 5:start + 5 + size].view((2,) + net.in_shape)
    plan._calls_for(odd)
    assert len(builds) == 4 and _flat(plan._calls) == _flat(build(plan, odd))


def test_refusals_name_the_call_that_moved():
    L = B.lib()
    f = B.fmt(4)
    empty = (L.dfq_quantize, (None, None, 0, f))
    conv = (L.dfq_conv_q, (1 << 20, 1 << 21, None, 1 << 22, None, 1, 8, 8, 4, 4, 1, 1, 1, 0, 1, 4, f, f, f, 1))
    calls = B.CallList([empty, conv], 1 << 20)
    moved = calls.rebind((1 << 22) + 16)                     # onto the result: refused before anything is launched
    assert moved[1][1][0] == (1 << 22) + 16 and conv[1][0] == 1 << 20
    with pytest.raises(B.DfqError, match="dfq_conv_q") as e:
        calls.run(None)
    assert e.value.status == B.EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["mobilenet", "fused", "codes", "np"])
def test_passes_on_tensors_in_turn(kind):
    from paper_1805_07941_amd import npnet
    rng = np.random.default_rng(8)
    if kind == "codes":
        net = _joined(True)
        xs = [torch.from_numpy(rng.integers(-127, 128, (2, 6, 6, 16)).astype(np.int8)).cuda() for _ in range(3)]
    else:
        net = wl.mobilenet_v1(batch=2, hw=64, classes=40) if kind == "mobilenet" else wl.resnet50(batch=2, hw=64, classes=40)
        xs = [torch.from_numpy(rng.standard_normal((2, 64, 64, 3)).astype(np.float32)).cuda() for _ in range(3)]
    if kind == "np":
        qz, _ = npnet.calibrate(net, xs[0])
        make = lambda: npnet.NpPlan(net, qz, 2)
    else:
        qz, _ = int8net.calibrate(net, xs[0])
        make = lambda: int8net.Plan(net, qz, 2, keep_all=kind == "codes", fuse=kind == "fused")
    want = []
    for x in xs:
        want.append(make().run(x).clone())
    assert not torch.equal(want[0], want[1])
    plan = make()
    for i in (0, 1, 2, 1, 0, 0):
        assert torch.equal(plan.run(xs[i]), want[i]), i
        assert torch.equal(plan.run_graph(xs[i]), want[i]) and torch.equal(plan.run_graph(xs[i]), want[i]), i
