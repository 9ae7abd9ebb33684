"""How calibration moves a network's float weights to the device: in groups of bounded size, every array with its own type and shape."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl
from paper_1805_07941_amd import net as int8net


def _net(bias_of=lambda b: b):
    net = wl.Net(3, "chain", 1, (8, 8, 4))
    net.shapes["input"] = net.in_shape
    t = net.conv("a", "input", 8, 3, pad=1)
    t = net.conv("b", t, 24, 1)
    t = net.conv("c", t, 16, 3, pad=1)
    net.output_name = net.conv("d", t, 5, 1)
    rng = np.random.default_rng(5)
    made = {nd.name: (rng.standard_normal((nd.K, nd.R, nd.R, net.shapes[nd.srcs[0]][2])).astype(np.float32), rng.standard_normal(nd.K).astype(np.float32))
            for nd in net.nodes if nd.op == "conv"}
    net.weights = lambda nd: (made[nd.name][0], bias_of(made[nd.name][1]))
    return net, made


@pytest.mark.parametrize("limit,groups", [(1 << 40, [4]), (0, [1, 1, 1, 1]), (4 * (8 * 36 + 24 * 8), [2, 1, 1]), (4 * (16 * 9 * 24 + 5 * 16), [2, 2])])
def test_groups(monkeypatch, limit, groups):
    net, made = _net()
    monkeypatch.setattr(int8net, "WEIGHT_GROUP_BYTES", limit)
    got = list(int8net.float_weights(net, "cpu", fold=False))
    assert [len(g) for g in got] == groups
    assert [n for g in got for n in g] == ["a", "b", "c", "d"]
    for g in got:
        assert len(g) == 1 or sum(4 * w.numel() for w, _ in g.values()) <= limit
        for name, (w, b) in g.items():
            assert np.array_equal(w.numpy(), made[name][0]) and np.array_equal(b.numpy(), made[name][1])


def test_bias_keeps_type_and_shape():
    """A bias that is no float32 vector is not turned into one by its neighbours: the conversion behind refuses what it refused."""
    net, made = _net(lambda b: b.astype(np.float64) if b.size == 24 else b)
    (g,) = int8net.float_weights(net, "cpu", fold=False)
    assert [b.dtype for _, b in g.values()] == [torch.float32, torch.float64, torch.float32, torch.float32]
    net, made = _net(lambda b: b.astype(np.float16) if b.size == 5 else b)
    (g,) = int8net.float_weights(net, "cpu", fold=False)
    assert g["d"][1].dtype == torch.float16
    net, made = _net(lambda b: b[:, None] if b.size == 8 else b)
    (g,) = int8net.float_weights(net, "cpu", fold=False)
    assert [tuple(b.shape) for _, b in g.values()] == [(8, 1), (24,), (16,), (5,)]


def test_no_convolutions():
    net = wl.Net(3, "none", 1, (8, 8, 4))
    assert list(int8net.float_weights(net, "cpu")) == []


@pytest.mark.gpu
@pytest.mark.parametrize("per_channel", [False, True])
def test_results_do_not_depend_on_the_groups(monkeypatch, per_channel):
    from paper_1805_07941_amd import npnet
    got = []
    for limit in (1 << 40, 0):
        monkeypatch.setattr(int8net, "WEIGHT_GROUP_BYTES", limit)
        net, _ = _net()
        x = torch.from_numpy(np.random.default_rng(6).standard_normal((2, 8, 8, 4)).astype(np.float32)).cuda()
        qz, t = int8net.calibrate(net, x, per_channel=per_channel)
        qn, tn = npnet.calibrate(net, x)
        got.append((qz, t, qn, tn))
    (qa, ta, na, xa), (qb, tb, nb, xb) = got
    assert qa.frac == qb.frac and na.frac == nb.frac and na.w_frac == nb.w_frac
    for name in qa.w:
        assert np.array_equal(qa.w_frac[name], qb.w_frac[name])
        assert torch.equal(qa.w[name], qb.w[name]) and torch.equal(qa.b[name], qb.b[name])
        assert torch.equal(na.w_codes[name], nb.w_codes[name]) and torch.equal(na.b[name], nb.b[name])
    for name in ta:
        assert torch.equal(ta[name], tb[name])
        assert all(torch.equal(u, v) for u, v in zip(xa[name], xb[name]))


@pytest.mark.parametrize("pieces", [1, 2, 4])
def test_a_pinned_piece_is_awaited_on_the_device_it_travels_to(monkeypatch, pieces):
    """Uploads to a device that is not the current one, with copies that happen as late as they may: when their stream is awaited."""
    empty, copy = torch.empty, torch.Tensor.copy_
    pending, waits = [], []

    class Stream:
        def __init__(self, device):
            self.device = str(device)

        def synchronize(self):
            waits.append(self.device)
            while pending:
                copy(*pending.pop(0))

    def late(dst, src, non_blocking=False):
        if not non_blocking:
            return copy(dst, src)
        pending.append((dst, src))
        return dst

    monkeypatch.setattr(torch, "empty", lambda *a, device=None, pin_memory=False, **kw: empty(*a, **kw))
    monkeypatch.setattr(torch.Tensor, "copy_", late)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    monkeypatch.setattr(int8net, "STAGING_BYTES", 4096)
    monkeypatch.setattr(int8net, "STAGING_PIECES", pieces)
    rng = np.random.default_rng(2)
    for sizes in ((700, 5, 3000, 64, 1023, 1, 2048), (1024,) * 8, (70000, 3), (1, 2, 3), (4096,), (1000, 1, 1023)):
        arrays = [rng.standard_normal(n).astype(np.float32) for n in sizes]
        got = int8net._to_device(arrays, "cuda:1")
        sent = sum(-(-n // 64) * 64 for n in sizes)
        assert waits == ["cuda:1"] * ((-(-sent // 1024) - 1) // pieces)           # none behind the last piece
        waits.clear()
        Stream("end").synchronize()
        waits.clear()
        assert all(np.array_equal(g.numpy(), a) for g, a in zip(got, arrays))


def test_pinned_pieces_of_an_upload(monkeypatch):
    """As many as an upload needs while it needs no wait; four where it waits in any case."""
    empty, pinned = torch.empty, []
    monkeypatch.setattr(torch, "empty", lambda *a, device=None, pin_memory=False, **kw: (pinned.append(a) if pin_memory else None, empty(*a, **kw))[1])
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: type("Stream", (), {"synchronize": lambda self: None})())
    monkeypatch.setattr(int8net, "STAGING_BYTES", 4096)
    for words, pieces in ((0, 1), (64, 1), (1024, 1), (1025, 2), (16 * 1024, 16), (16 * 1024 + 1, 4), (100 * 1024, 4)):
        a = np.arange(words, dtype=np.float32)
        (got,) = int8net._to_device([a], "cuda:0")
        assert len(pinned) == pieces and np.array_equal(got.numpy(), a)
        pinned.clear()
