"""What a call keeps of the layers it has met (descriptor, shape of the result, bytes of scratch) goes by their numbers, whatever holds these."""
import numpy as np
import pytest
import torch

from paper_1412_4564_amd import binding as B

XS, WS = (2, 16, 20, 24), (40, 16, 3, 3)
HOLD = {"tensors": lambda *v: [torch.tensor(n) for n in v], "arrays": lambda *v: [np.array(n) for n in v], "scalars": lambda *v: np.array(v)}


@pytest.mark.parametrize("hold", sorted(HOLD))
def test_numbers_that_change_in_place(hold):
    two, four = HOLD[hold](1, 1), HOLD[hold](1, 1, 1, 1)
    calls = (lambda: B._conv(XS, WS, two, four, B.MCN_PREC_FP32, B.MCN_OP_FORWARD),
             lambda: B._convt(XS, (16, 8, 4, 4), two, four, 1, B.MCN_PREC_FP32, B.MCN_OP_FORWARD),
             lambda: B._pool(XS, (3, 3), two, four, B.MCN_POOL_MAX, True))
    fresh = (lambda s, p: B.make_desc(XS, WS, s, p), lambda s, p: B.make_convt_desc(XS, (16, 8, 4, 4), s, p), lambda s, p: B.make_pool_desc(XS, (3, 3), s, p))
    for s, p in (((1, 1), (1, 1, 1, 1)), ((2, 1), (1, 1, 1, 1)), ((2, 3), (0, 1, 2, 1))):
        for i in range(2):
            two[i] += s[i] - int(two[i])           # in place: the same objects with other numbers
        for i in range(4):
            four[i] += p[i] - int(four[i])
        for call, f in zip(calls, fresh):
            assert bytes(call()[0]) == bytes(f(s, p))


def test_shapes_in_any_sequence():
    want = B._conv(XS, WS, (2, 1), (1, 0, 1, 0), B.MCN_PREC_FP32, B.MCN_OP_FORWARD)
    for hold in (list, np.array, torch.Size, lambda v: [np.int64(n) for n in v]):
        got = B._conv(hold(XS), hold(WS), [2, 1], [1, 0, 1, 0], B.MCN_PREC_FP32, B.MCN_OP_FORWARD)
        assert bytes(got[0]) == bytes(want[0]) and got[1:] == want[1:]


@pytest.mark.gpu
def test_filter_and_bias_outputs_come_both():
    x, p = torch.ones(XS, device="cuda"), torch.ones(2, 40, 18, 22, device="cuda")
    out = torch.empty(WS, device="cuda"), torch.empty(40, device="cuda")
    print("outputs of the filter and bias derivative", flush=True)
    got = B.conv_backward_filter_bias(x, WS, p, out=out)
    assert got[0] is out[0] and got[1] is out[1] and torch.equal(got[1], torch.full_like(got[1], 2.0 * 22 * 18))
    for bad in ((None, out[1]), (out[0], None)):
        with pytest.raises(TypeError):
            B.conv_backward_filter_bias(x, WS, p, out=bad)
