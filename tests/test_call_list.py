"""A pass as one library call: records against the functions they stand for."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")

from paper_1805_07941_amd import binding as B


def test_records_reach_their_functions():
    """Calls that are refused before anything is launched: each by its own function, the first refusal ends the list."""
    L = B.lib()
    bad_fmt, f = B.fmt(99), B.fmt(4)
    conv = (1 << 20, 1 << 21, None, 1 << 22, None, 1, 8, 8, 4, 4, 1, 1, 1, 0, 1, 4)
    empty = (L.dfq_quantize, (None, None, 0, f))                                # nothing to do: accepted
    cases = [((L.dfq_quantize, (1 << 20, 1 << 21, 8, bad_fmt)), B.EFMT),
             ((L.dfq_conv_q, conv + (bad_fmt, f, f, 1)), B.EFMT),
             ((L.dfq_conv_q, conv[:5] + (1, 0, 8, 4, 4, 1, 1, 1, 0, 1, 4) + (f, f, f, 1)), B.ESHAPE),
             ((L.dfq_pool_q, (1 << 20, 1 << 21, 7, 1, 8, 8, 4, 2, 2, 0, f, f)), B.EINVAL),
             ((L.dfq_concat_q_into, (0, (C.c_void_p * 1)(), (C.c_int * 1)(), (B.Fmt * 1)(), 1 << 20, 4, f, 1)), B.EINVAL),
             ((L.dfq_conv_np, (1 << 20, 1 << 21, 1 << 22, 1 << 23, None, None, None, None, 1, 8, 8, 64, 16, 1, 1, 1, 0, 1, 0, 0, 0, 4, 0)), B.EINVAL),
             ((L.dfq_stem_pack_x, (1 << 20, 1 << 21, 1, 8, 8, 9, 3, 3, 1)), None)]
    for call, status in cases:
        direct = call[0](*call[1], None)
        assert direct != B.OK and status in (None, direct)
        with pytest.raises(B.DfqError, match=call[0].__name__) as e:
            B.CallList([empty, call, empty]).run(None)
        assert e.value.status == direct
    B.CallList([empty, empty]).run(None)
    B.CallList([]).run(None)


def test_every_plan_call_has_a_number():
    """What the plans issue: a call that the list does not know is refused, never skipped."""
    import re
    import paper_1805_07941_amd.net as net, paper_1805_07941_amd.npnet as npnet
    L = B.lib()
    for module in (net, npnet):
        body = open(module.__file__).read()
        body = body[body.index("def _build_calls"):]
        for name in sorted(set(re.findall(r"L\.(dfq_\w+)", body))):
            assert L.dfq_call_number(name.encode()) >= 0, name
    assert L.dfq_call_number(b"dfq_absmax_f32") == -1 and L.dfq_call_number(None) == -1
    with pytest.raises(B.DfqError):
        B.CallList([(L.dfq_absmax_f32, (None, 0, None))]).run(None)
    with pytest.raises(B.DfqError):
        B.CallList([(L.dfq_quantize, (None, None, 0))]).run(None)               # an argument is missing
