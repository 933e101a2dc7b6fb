"""1x1 filters and fully-connected layers on the bf16 matrix core with operands in three bf16 planes (kern_igemm_split.h, units of several
channel groups): every result against the oracle at the edges of tiles, images and units, and values that a split operand cannot carry."""
import numpy as np
import pytest
import torch

import oracle
import parity_util as U
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth
from test_gpu_parity import custom_layer

pytestmark = pytest.mark.gpu

# n terms are off by at most n/4 * 2^-25 of the sum of |w||x|, with random signs by about sqrt(n/4) * 2^-25 (an MFMA rounds four times
# in 16 terms): 1e-6 for the largest n here, 1200.  5e-6 leaves a factor 5.
BOUND = 5e-6

CASES = [  # H, W, D, N, Hf, Wf, Df, K, stride, pad
    (7, 7, 500, 16, 1, 1, 500, 250, (1, 1), (0, 0, 0, 0)),       # tiles across images, last unit of few channels
    (30, 31, 200, 10, 1, 1, 200, 96, (2, 2), (0, 0, 0, 0)),      # strided forward, 13 groups in units of as many as fit
    (45, 15, 87, 8, 1, 1, 87, 64, (1, 1), (0, 0, 0, 0)),         # odd channels, 64 filters
    (16, 40, 240, 19, 1, 1, 120, 494, (1, 1), (0, 0, 0, 0)),     # two groups of filters, 247 each
    (13, 12, 144, 30, 1, 1, 144, 100, (1, 1), (1, 0, 2, 1)),     # pads: pixels that read nothing
    (9, 9, 70, 40, 1, 1, 70, 30, (1, 1), (0, 0, 0, 0)),          # tiles of 32 filters
    (24, 40, 344, 5, 1, 1, 344, 144, (1, 1), (0, 0, 0, 0)),      # 225 tiles of dzdx
    (36, 12, 500, 16, 1, 1, 500, 160, (1, 1), (0, 0, 0, 0)),     # shared tiles
    (5, 5, 131, 37, 5, 5, 131, 701, (1, 1), (0, 0, 0, 0)),       # fully connected, everything odd
    (4, 4, 96, 130, 4, 4, 96, 1100, (1, 1), (0, 0, 0, 0)),
    (1, 1, 248, 168, 1, 1, 248, 1200, (1, 1), (0, 0, 0, 0)),
]


def run(L, x, w, b, p, precision=B.MCN_PREC_FP32):
    st, pad = L["stride"], L["pad"]
    out = {"y": B.conv_forward(x, w, b, st, pad, precision), "dzdx": B.conv_backward_data(x.shape, w, p, st, pad, precision)}
    if L["Hf"] == L["H"]:
        out["dzdw"] = B.conv_backward_filter(x, w.shape, p, st, pad, precision)
    return out


def sums(L, x, w, b, p):
    st, pad = L["stride"], L["pad"]
    return {"y": oracle.forward(x, w, b, st, pad), "dzdx": oracle.backward_data(x.shape, w, p, st, pad),
            "dzdw": oracle.backward_filter(x, w.shape, p, st, pad) if L["Hf"] == L["H"] else None}


def planes(L, precision=B.MCN_PREC_FP32):
    d = B.make_desc(synth.x_shape(L), synth.w_shape(L), L["stride"], L["pad"], precision)
    return [B.mcn_conv_operand_planes(d, op) for op in (B.MCN_OP_FORWARD, B.MCN_OP_BACKWARD_DATA, B.MCN_OP_BACKWARD_FILTER)]


def inputs(L, seed):
    x, w, b = synth.make_x(L, seed), synth.make_w(L, seed), synth.make_b(L, seed)
    return x, w, b, synth.make_dzdy(L, *oracle.output_size(x.shape, w.shape, L["stride"], L["pad"]), seed)


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_every_result(case, misalign):
    L = custom_layer(*CASES[case], idx=920 + case)
    assert 3 in planes(L)[:2] and planes(L, B.MCN_PREC_FP32_PLAIN) == [0, 0, 0]
    host = inputs(L, case)
    dev = [U.gpu(t, misalign) for t in host]
    got = run(L, *dev)
    ref, den = sums(L, *(U.np64(t) for t in host)), sums(L, *(np.abs(U.np64(t)) for t in host))
    for name in got:
        e = U.norm_err(got[name].cpu().numpy(), ref[name], den[name])
        print("pointwise in three planes", case, misalign, name, e, flush=True)
        assert e <= BOUND
    again = run(L, *dev)
    assert all(torch.equal(got[name], again[name]) for name in got)
    assert torch.equal(B.conv_relu_forward(dev[0], dev[1], dev[2], L["stride"], L["pad"]), got["y"].clamp(min=0.0))


@pytest.mark.parametrize("case", [0, 1, 4, 7, 8, 10])
def test_values_that_are_not_finite(case):
    """Results that meet an infinity or a NaN are those of the plain sum, all others as without them."""
    L = custom_layer(*CASES[case], idx=940 + case)
    x, w, b, p = inputs(L, 3)
    clean = run(L, x.cuda(), w.cuda(), b.cuda(), p.cuda())
    mark = lambda t, at, v: t.view(-1).__setitem__(at, v)
    marks = [torch.zeros_like(t) for t in (x, w, p)]
    # x of the first pixel, the last weight, the last dzdy: read by stride 2 too
    mark(x, 0, float("inf")); mark(w, w.numel() - 1, float("nan")); mark(p, p.numel() - 1, float("-inf"))
    mark(marks[0], 0, 1.0); mark(marks[1], w.numel() - 1, 1.0); mark(marks[2], p.numel() - 1, 1.0)
    got, want = run(L, x.cuda(), w.cuda(), b.cuda(), p.cuda()), sums(L, *(U.np64(t) for t in (x, w, b, p)))
    ones = [np.ones(t.shape) for t in (x, w, p)]
    mx, mw, mp = (U.np64(t) for t in marks)
    a, c = sums(L, mx, ones[1], None, mp), sums(L, ones[0], mw, None, ones[2])
    touched = {"y": a["y"] + c["y"] > 0, "dzdx": sums(L, ones[0], ones[1], None, mp)["dzdx"] + c["dzdx"] > 0}
    if "dzdw" in got:
        touched["dzdw"] = sums(L, mx, ones[1], None, ones[2])["dzdw"] + sums(L, ones[0], ones[1], None, mp)["dzdw"] > 0
    for name in got:
        t, g = torch.from_numpy(np.asarray(touched[name])).reshape(got[name].shape), got[name].cpu()
        r = torch.from_numpy(np.asarray(want[name])).reshape(g.shape)
        assert t.any() and torch.equal(g[~t], clean[name].cpu()[~t])
        assert torch.equal(torch.isnan(g[t]), torch.isnan(r[t])) and torch.equal(g[t][torch.isinf(r[t])].double(), r[t][torch.isinf(r[t])])


@pytest.mark.parametrize("case", range(len(CASES)))
def test_results_summed_again(case):
    """Operands that round to infinity in their first plane, where the other operand is tiny: every result that they enter is summed again, to
    one of ordinary size, in which no term may be missing or count twice."""
    L = custom_layer(*CASES[case], idx=960 + case)
    assert 3 in planes(L)[:2]
    x, w, b, p = inputs(L, 6)
    # Per pass, so that no result consists of products of two tiny numbers, which fp32 does not hold.
    large = {"y": [t.clone() for t in (x, w, b, p)], "dzdx": [t.clone() for t in (x, w, b, p)], "dzdw": [t.clone() for t in (x, w, b, p)]}
    t = large["y"]; t[0][0, 1, 0, 0] = 3.4e38; t[1][:, 1, 0, 0] *= 1e-37
    t = large["dzdx"]; t[3][-1, -1, 0, 0] = 3.4e38; t[1][-1] *= 1e-37
    t = large["dzdw"]; t[0][0, 1, 0, 0] = t[3][-1, -1, 0, 0] = 3.4e38; t[3][0] *= 1e-37; t[0][-1] *= 1e-37
    for name, t in large.items():
        ref, den = sums(L, *(U.np64(v) for v in t))[name], sums(L, *(np.abs(U.np64(v)) for v in t))[name]
        if ref is None:
            continue
        e = U.norm_err(run(L, *(v.cuda() for v in t))[name].cpu().numpy(), ref, den)
        print("pointwise, summed again", case, name, e, flush=True)
        assert e <= BOUND
