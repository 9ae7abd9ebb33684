"""The work a user of this framework has it do, as cases that can be timed and compared.

Six kinds, every one through the public entry points:

* ``net``        one pass of a calibrated network in int8 (``net.Plan``), eager or replayed from a graph;
* ``np``         the same on (8, p) dynamic floating-point codes (``npnet.NpPlan``);
* ``calibrate``  choosing the formats of a network from one batch (``net.calibrate``);
* ``np_calibrate``  the same for (8, p) codes (``npnet.calibrate``);
* ``layer``      one convolution of a user's own network (``conv_q``, ``conv_q_pc``), any geometry;
* ``stream``     the layers between convolutions, one by one (``quantize``, ``pool_q``, ``eltwise_q``, ``concat_q``, ``dequantize``).

Weights and images have the statistics of the synthetic workloads (He-normal weights, N(0, 0.1) bias, N(0, 1) images)."""
import math

import numpy as np
import torch

import workloads as wl
from paper_1805_07941_amd import binding as B
from paper_1805_07941_amd import net as int8net
from paper_1805_07941_amd import npnet

DEV = "cuda:0"


def listed():
    return [
        # the benchmark's workload: bulk classification of 224 x 224 images, formats per layer
        dict(name="resnet50_b256", kind="net", net="resnet50", batch=256, hw=224, classes=1000, per_channel=False, graph=True),
        # one image at a time, as an online service answers it
        dict(name="resnet50_b1", kind="net", net="resnet50", batch=1, hw=224, classes=1000, per_channel=False, graph=True),
        # the paper's own rule (a weight format per output channel), images of an odd size, a batch that fills no tile, eager calls
        dict(name="resnet50_pc_b12_hw201", kind="net", net="resnet50", batch=12, hw=201, classes=1000, per_channel=True, graph=False),
        # the depthwise-separable network at its batch of the configurations
        dict(name="mobilenet_b128", kind="net", net="mobilenet_v1", batch=128, hw=224, classes=1000, per_channel=False, graph=True),
        # the same for one image by eager calls: the smallest pass, mostly launches
        dict(name="mobilenet_b1", kind="net", net="mobilenet_v1", batch=1, hw=224, classes=1000, per_channel=False, graph=False),
        # a block of branches joined by concat, from int8 codes
        dict(name="inception_b64", kind="net", net="inception", batch=64, hw=28, classes=0, per_channel=False, graph=True),
        # bulk classification on the format the paper reports as the most accurate
        dict(name="resnet50_np84_b64", kind="np", blocks="3463", batch=64, hw=224, classes=1000, p=4, graph=True),
        # formats of a network from a calibration batch of 8 images (the paper takes 8 to 128), per output channel
        dict(name="calibrate_mobilenet_b8", kind="calibrate", net="mobilenet_v1", batch=8, hw=224, classes=1000, per_channel=True, rule="maxabs"),
        # the same on (8, 4) codes for a residual network with one block per stage
        dict(name="np_calibrate_residual_b4", kind="np_calibrate", blocks="1111", batch=4, hw=160, classes=200, p=4),
        # a dense layer whose channel counts (pruned networks) and image sides are multiples of nothing
        dict(name="layer_ragged_3x3", kind="layer", N=16, H=57, W=43, C=83, K=131, R=3, stride=1, groups=1, per_channel=False, relu=True),
        # a grouped layer of the benchmark's set
        dict(name="layer_grouped_28_256", kind="layer", N=64, H=28, W=28, C=256, K=256, R=3, stride=1, groups=32, per_channel=False, relu=True),
        # what stands between convolutions, over tensors with a ragged number of channels
        dict(name="stream_ragged", kind="stream", N=24, H=45, W=61, C=90, k=3, relu=True),
    ]


def _spread(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["net", "np", "calibrate", "np_calibrate", "layer", "stream"], [30, 10, 10, 8, 26, 16])[0]
    if kind == "net":
        name = rng.choice(["resnet50", "resnet50", "mobilenet_v1", "inception"])
        if name == "inception":
            return dict(kind=kind, net=name, batch=_spread(rng, 1, 128), hw=rng.randint(9, 36), classes=0, per_channel=rng.random() < 0.5,
                        graph=rng.random() < 0.5)
        hw = rng.choice([224, rng.randint(80, 256), 32 * rng.randint(3, 8)])
        most = max(1, min(256, 256 * 224 * 224 // (hw * hw)))
        return dict(kind=kind, net=name, batch=_spread(rng, 1, most), hw=hw, classes=rng.choice([1000, rng.randint(10, 1000)]),
                    per_channel=rng.random() < 0.4, graph=rng.random() < 0.5)
    if kind == "np":
        return dict(kind=kind, blocks=rng.choice(["1111", "3463"]), batch=_spread(rng, 1, 64), hw=rng.choice([224, rng.randint(80, 224)]),
                    classes=rng.choice([1000, rng.randint(10, 1000)]), p=rng.choice([4, 4, 5, 7]), graph=rng.random() < 0.5)
    if kind == "calibrate":
        name = rng.choice(["mobilenet_v1", "inception"])
        per_channel = rng.random() < 0.5
        return dict(kind=kind, net=name, batch=_spread(rng, 2, 24), hw=rng.randint(9, 32) if name == "inception" else rng.randint(96, 224),
                    classes=rng.choice([1000, rng.randint(10, 1000)]), per_channel=per_channel,
                    rule="maxabs" if per_channel or rng.random() < 0.7 else "search")
    if kind == "np_calibrate":
        return dict(kind=kind, blocks="1111", batch=_spread(rng, 1, 4), hw=rng.randint(80, 160), classes=rng.randint(10, 400), p=rng.choice([4, 4, 5, 7]))
    if kind == "layer":
        R = rng.choice([1, 3, 3, 5])
        stride = rng.choice([1, 1, 2])
        style = rng.choice(["dense", "dense16", "ragged", "grouped", "depthwise"])
        if style == "dense":
            groups, C, K = 1, 64 * _spread(rng, 1, 16), 64 * _spread(rng, 1, 16)
        elif style == "dense16":
            groups, C, K = 1, 16 * _spread(rng, 1, 24), _spread(rng, 8, 384)
        elif style == "ragged":
            groups, C, K = 1, _spread(rng, 5, 320), _spread(rng, 8, 320)
        elif style == "grouped":
            groups = rng.choice([2, 4, 8, 16, 32])
            C, K = groups * _spread(rng, 3, 16), groups * _spread(rng, 3, 16)
        else:
            R = 3
            C = K = groups = rng.choice([16 * _spread(rng, 2, 40), _spread(rng, 24, 640)])
        H, W = _spread(rng, 7, 80), _spread(rng, 7, 80)
        macs = (H // stride) * (W // stride) * K * R * R * (C // groups)
        most = max(1, min(256, int(8e9 // macs), int(120e6 // (H * W * (C + K // (stride * stride))))))
        return dict(kind=kind, N=_spread(rng, 1, most), H=H, W=W, C=C, K=K, R=R, stride=stride, groups=groups,
                    per_channel=rng.random() < 0.3, relu=rng.random() < 0.7)
    H, W, C = _spread(rng, 7, 112), _spread(rng, 7, 112), _spread(rng, 3, 512)
    return dict(kind=kind, N=_spread(rng, 1, max(1, min(128, int(12e6 // (H * W * C))))), H=H, W=W, C=C, k=rng.choice([2, 3, 3, 5]), relu=rng.random() < 0.5)


def tolerance(case):
    # every result is an integer sum rounded once by a stated rule, so two correct implementations agree in every bit; the logits
    # are int8 codes (or (8, p) codes) times a power of two, exact in float
    return "exact"


# ---- networks ------------------------------------------------------------------------------- #
def _residual(batch, hw, classes, blocks):
    """The residual network of the workloads with its own number of blocks per stage."""
    if blocks == "3463":
        return wl.resnet50(batch=batch, hw=hw, classes=classes)
    net = wl.Net(4, "residual", batch, (hw, hw, 3))
    net.shapes["input"] = net.in_shape
    t = net.conv("stem", "input", 64, 7, stride=2, pad=3)
    t = net.pool("maxpool", "pool1", t, 3, 2, pad=1)
    for si, (count, width) in enumerate(zip([int(c) for c in blocks], [64, 128, 256, 512]), start=2):
        for bi in range(count):
            st = 2 if (bi == 0 and si > 2) else 1
            pre = "s%db%d" % (si, bi)
            a = net.conv(pre + "_a", t, width, 1)
            b = net.conv(pre + "_b", a, width, 3, stride=st, pad=1)
            c = net.conv(pre + "_c", b, 4 * width, 1, relu=False)
            sc = net.conv(pre + "_proj", t, 4 * width, 1, stride=st, relu=False) if bi == 0 else t
            t = net.eltwise(pre + "_add", c, sc, relu=True)
    t = net.pool("avgpool", "gap", t, net.shapes[t][0], 1)
    net.output_name = net.conv("fc", t, classes, 1, relu=False)
    return net


def _graph_of(case):
    if case["kind"] in ("np", "np_calibrate"):
        return _residual(case["batch"], case["hw"], case["classes"], case["blocks"])
    if case["net"] == "inception":
        return wl.inception_block(batch=case["batch"], hw=case["hw"])
    return getattr(wl, case["net"])(batch=case["batch"], hw=case["hw"], classes=case["classes"])


def _weights(net, gen):
    """The float weights a user loads: host arrays, drawn on the device from the seed."""
    made = {}
    for nd in net.nodes:
        if nd.op == "conv":
            cg = net.shapes[nd.srcs[0]][2] // nd.groups
            w = torch.randn((nd.K, nd.R, nd.R, cg), generator=gen, device=DEV) * math.sqrt(2.0 / (nd.R * nd.R * cg))
            b = torch.randn((nd.K,), generator=gen, device=DEV) * 0.1
            made[nd.name] = (w.cpu().numpy(), b.cpu().numpy())
    net.weights = lambda nd: made[nd.name]


def _codes(shape, gen, scale):
    return torch.round(torch.randn(shape, generator=gen, device=DEV) * scale).clamp_(-127, 127).to(torch.int8)


def _images(net, batch, gen):
    if net.input_is_int8:
        return _codes((batch,) + tuple(net.in_shape), gen, 2.0 ** net.f_input_codes)
    return torch.randn((batch,) + tuple(net.in_shape), generator=gen, device=DEV)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind in ("net", "np", "calibrate", "np_calibrate"):
        net = _graph_of(case)
        _weights(net, gen)
        x = _images(net, case["batch"], gen)
        st = dict(case=case, net=net, x=x)
        some = x[: min(4, case["batch"])].contiguous()
        if kind == "net":
            qz, _ = int8net.calibrate(net, some, keep_tensors=False, per_channel=case["per_channel"])
            # the block of branches keeps all of its tensors (what a user looks at is the joined one), the others reuse buffers
            st["plan"] = (int8net.Plan(net, qz, case["batch"]) if case["net"] == "inception"
                          else int8net.Plan(net, qz, case["batch"], keep_all=False, fuse=True))
        elif kind == "np":
            qz, _ = npnet.calibrate(net, x[:1].contiguous(), p=case["p"])
            st["plan"] = npnet.NpPlan(net, qz, case["batch"])
        return st
    if kind == "layer":
        N, H, W, C, K, R, g = (case[k] for k in ("N", "H", "W", "C", "K", "R", "groups"))
        x = _codes((N, H, W, C), gen, 24.0)
        w = _codes((K, R, R, C // g), gen, 36.0)
        b = torch.randint(-20000, 20001, (K,), generator=gen, device=DEV, dtype=torch.int32)
        # the rescale a calibration would choose: the outputs' spread is about 30 codes
        shift = max(0, int(round(math.log2(math.sqrt(R * R * (C // g)) * 24 * 36 / 30))))
        st = dict(case=case, x=x, w=w, b=b, f_in=4, f_out=4, f_w=shift)
        if case["per_channel"]:
            f_w = torch.randint(max(0, shift - 1), shift + 2, (K,), generator=gen, device=DEV, dtype=torch.int32)
            st["f_w"], st["f_w_range"] = f_w, (int(f_w.min()), int(f_w.max()))
        return st
    shape = tuple(case[k] for k in ("N", "H", "W", "C"))
    return dict(case=case, x=torch.randn(shape, generator=gen, device=DEV), other=_codes(shape, gen, 30.0))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("net", "np"):
        plan = state["plan"]
        out = plan.run_graph(state["x"]) if case["graph"] else plan.run(state["x"])
        if kind == "net" and case["net"] == "inception":
            return {"codes": plan.buf[state["net"].output_name], "values": out}
        return out
    if kind == "calibrate":
        net = state["net"]
        qz, t = int8net.calibrate(net, state["x"], keep_tensors=False, per_channel=case["per_channel"], rule=case["rule"])
        return {"frac": np.array(list(qz.frac.values())), "w_frac": np.concatenate([np.atleast_1d(v) for v in qz.w_frac.values()]),
                "w": list(qz.w.values()), "b": list(qz.b.values()), "out": t[net.output_name]}
    if kind == "np_calibrate":
        net = state["net"]
        qz, t = npnet.calibrate(net, state["x"], p=case["p"])
        return {"frac": np.array(list(qz.frac.values())), "w_frac": np.array(list(qz.w_frac.values())), "w": list(qz.w.values()),
                "b": list(qz.b.values()), "out": t[net.output_name]}
    if kind == "layer":
        pad = case["R"] // 2
        if case["per_channel"]:
            y, _ = B.conv_q_pc(state["x"], state["w"], state["b"], state["f_in"], state["f_w"], state["f_out"], case["stride"], pad,
                               case["groups"], case["relu"], frac_w_range=state["f_w_range"])
        else:
            y, _ = B.conv_q(state["x"], state["w"], state["b"], state["f_in"], state["f_w"], state["f_out"], case["stride"], pad,
                            case["groups"], case["relu"])
        return y
    k = case["k"]
    q = B.quantize(state["x"], 5)
    same = B.pool_q(q, "max", 3, 1, 1, 5, 5)                              # a pooling branch keeps the image's size
    s, _ = B.eltwise_q(q, 5, state["other"], 4, 4, case["relu"])
    c = B.concat_q([same, s, state["other"]], [5, 4, 4], 4)
    m = B.pool_q(c, "max", k, 2, k // 2, 4, 4)
    a = B.pool_q(c, "avg", k, k, 0, 4, 5)
    return {"q": q, "same": same, "sum": s, "joined": c, "max": m, "avg": a, "values": B.dequantize(m, 4)}


# ---- the least work of a pass ----------------------------------------------------------------- #
def _net_work(net, batch, x_bytes, planes):
    """Every tensor that is stored between two kernels written once and read once per reader; joins and the pooling behind the
    first layer taken where their operand is produced."""
    size = lambda name: batch * math.prod(net.shapes[name]) * planes
    fused = {nd.srcs[0] for nd in net.nodes if nd.op == "eltwise"} | {nd.srcs[0] for nd in net.nodes if nd.op == "maxpool" and nd.stride == 2}
    total = batch * math.prod(net.in_shape) * x_bytes + batch * math.prod(net.shapes[net.output_name]) * 4
    for nd in net.nodes:
        total += sum(size(s) for s in nd.srcs if s not in fused and s != net.input_name)
        if nd.op == "concat":
            total -= sum(size(s) for s in nd.srcs) + size(nd.dst)         # branches can be written in place
        if nd.dst not in fused:
            total += size(nd.dst)
        if nd.op == "conv":
            cg = net.shapes[nd.srcs[0]][2] // nd.groups
            total += nd.K * nd.R * nd.R * cg * planes + 4 * nd.K
    return {"bytes": total, "flops": 2 * batch * net.macs_per_image()}


def work(case):
    kind = case["kind"]
    if kind == "net":
        net = _graph_of(case)
        return _net_work(net, case["batch"], 1 if net.input_is_int8 else 4, 1)
    if kind == "np":
        return _net_work(_graph_of(case), case["batch"], 4, 2)
    if kind in ("calibrate", "np_calibrate"):
        # a layer's output format depends on all of its sums, so they are formed, and what is stored is the calibrated tensors;
        # the float weights come from the host once and are read twice (maximum, conversion)
        net = _graph_of(case)
        planes = 1 if kind == "calibrate" else 2
        w = _net_work(net, case["batch"], 1 if net.input_is_int8 else 4, planes)
        w["bytes"] += sum(8 * nd.K * (nd.R * nd.R * (net.shapes[nd.srcs[0]][2] // nd.groups) + 1) for nd in net.nodes if nd.op == "conv")
        return w
    N, H, W, C = (case[k] for k in ("N", "H", "W", "C"))
    if kind == "layer":
        K, R, st = case["K"], case["R"], case["stride"]
        P, Q = wl.out_dim(H, R, st, R // 2), wl.out_dim(W, R, st, R // 2)
        wsize = K * R * R * (C // case["groups"])
        return {"bytes": N * H * W * C + N * P * Q * K + wsize + 4 * K, "flops": 2 * N * P * Q * wsize}
    k, n = case["k"], N * H * W * C
    pooled = N * wl.out_dim(H, k, 2, k // 2) * wl.out_dim(W, k, 2, k // 2) * 3 * C
    means = N * (H // k) * (W // k) * 3 * C
    # quantize 4 + 1, pooling 1 + 1, add 2 + 1, concat 3 + 3, two poolings 3 each and their results, dequantize 1 + 4 per pooled value
    return {"bytes": n * (5 + 2 + 3 + 6 + 6) + pooled * (1 + 1 + 4) + means, "flops": n * (1 + 9 + 1 + 6 * k * k)}
