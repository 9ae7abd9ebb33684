"""Which kernel a call launches, read from the device's own activity records: a variant asked for by name runs that kernel and no
other, at every size, and an automatic call runs the one that conv_q_select names."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_ops import B             # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

# the kernels' names in the compiled library
KERNEL_OF = {"MFMA": ("conv_mfma_kernel",), "POINTWISE": ("conv_pw_kernel",), "SPLIT": ("conv_sk_kernel",), "RAGGED": ("conv_rag_kernel",),
             "DIRECT": ("conv_direct_kernel",), "DEPTHWISE": ("conv_depthwise_kernel", "conv_dwm_"), "SMALLC": ("conv_smallc_", "conv_stem_"),
             "GROUPED": ("conv_grouped_kernel", "conv_sg_kernel")}


def launched(calls):
    """Names of the library's convolution kernels that each of the calls launched, in order."""
    calls[0]()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        for call in calls:
            call()
        torch.cuda.synchronize()
    events = [e for e in prof.events() if e.device_type == torch.autograd.DeviceType.CUDA and "conv_" in e.name]
    if not events:
        pytest.skip("the device's activity is not recorded here")
    return [e.name for e in sorted(events, key=lambda e: e.time_range.start)]


def operands(N, H, W, C, K, R, groups):
    x = torch.randint(-128, 128, (N, H, W, C), dtype=torch.int8, device="cuda")
    w = torch.randint(-128, 128, (K, R, R, C // groups), dtype=torch.int8, device="cuda")
    return x, w, torch.randint(-1000, 1000, (K,), dtype=torch.int32, device="cuda")


def test_named_variant_runs_its_kernel(B):
    cases = [("MFMA", (1, 14, 14, 256, 256, 3, 1, 1, 1)), ("MFMA", (2, 20, 20, 64, 128, 3, 1, 1, 1)), ("MFMA", (8, 1, 1, 512, 100, 1, 1, 0, 1)),
             ("MFMA", (1, 1, 1, 64, 80, 1, 1, 0, 1)), ("SPLIT", (1, 14, 14, 256, 256, 3, 1, 1, 1)), ("SPLIT", (40, 40, 40, 64, 64, 1, 1, 0, 1)),
             ("POINTWISE", (1, 14, 14, 256, 512, 1, 1, 0, 1)), ("RAGGED", (1, 14, 14, 64, 64, 3, 1, 1, 1)), ("DIRECT", (1, 14, 14, 64, 64, 3, 1, 1, 1))]
    calls = []
    for name, (N, H, W, C, K, R, st, pad, g) in cases:
        ops = operands(N, H, W, C, K, R, g)
        calls.append(lambda ops=ops, st=st, pad=pad, g=g, v=getattr(B, "CONV_" + name): B.conv_q(*ops, 4, 8, 4, st, pad, g, True, variant=v))
    got = launched(calls)
    assert len(got) == len(cases), got
    for (name, shape), kernel in zip(cases, got):
        assert any(k in kernel for k in KERNEL_OF[name]), (name, shape, kernel)


def test_select_names_what_an_automatic_call_runs(B):
    shapes = [(1, 56, 56, 64, 64, 3, 1, 1, 1), (48, 56, 56, 64, 64, 3, 1, 1, 1), (1, 7, 7, 512, 2048, 1, 1, 0, 1), (64, 7, 7, 512, 2048, 1, 1, 0, 1),
              (24, 28, 28, 128, 512, 1, 1, 0, 1), (1, 28, 28, 128, 512, 1, 1, 0, 1), (12, 56, 56, 256, 64, 1, 1, 0, 1), (12, 56, 56, 64, 256, 1, 1, 0, 1),
              (1, 14, 14, 64, 256, 1, 1, 0, 1), (16, 28, 28, 192, 384, 1, 1, 0, 1), (16, 28, 28, 192, 100, 1, 1, 0, 1), (4, 28, 28, 96, 100, 3, 2, 1, 1),
              (2, 20, 20, 83, 131, 3, 1, 1, 1), (2, 20, 20, 3, 40, 3, 2, 1, 1), (2, 20, 20, 64, 64, 3, 1, 1, 64), (2, 20, 20, 20, 30, 3, 1, 1, 5),
              (2, 20, 20, 15, 10, 3, 1, 1, 5), (2, 20, 20, 26, 26, 3, 1, 1, 26)]
    calls = []
    for (N, H, W, C, K, R, st, pad, g) in shapes:
        ops = operands(N, H, W, C, K, R, g)
        calls.append(lambda ops=ops, st=st, pad=pad, g=g: B.conv_q(*ops, 4, 8, 4, st, pad, g, True))
    got = launched(calls)
    assert len(got) == len(shapes), got
    seen = set()
    for (N, H, W, C, K, R, st, pad, g), kernel in zip(shapes, got):
        name = B.CONV_VARIANT_NAMES[B.conv_q_select(N, H, W, C, K, R, R, st, pad, g)].upper()
        seen.add(name)
        assert any(k in kernel for k in KERNEL_OF[name]), (name, (N, H, W, C, K, R, st, pad, g), kernel)
    assert len(seen) == 8, seen
