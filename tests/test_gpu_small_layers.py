"""Small fp32 layers (csrc/kern_small.h), where a pass is one launch: every element against the oracle at the edges of its blocks (64 pixels, 8
filters, eight shares of the reduction, 256 and 1024 pixels of the filter derivative) and just beyond its limits, where the tile kernels take over."""
import pytest
import torch

import oracle
import parity_util as U
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth

pytestmark = pytest.mark.gpu


def layer(H, W, D, N, Hf, Wf, Df, K, stride, pad, idx=0):
    return dict(H=H, W=W, D=D, N=N, Hf=Hf, Wf=Wf, Df=Df, K=K, stride=stride, pad=pad, config=23, index=idx)


CASES = [  # H, W, D, N, Hf, Wf, Df, K, stride, pad
    (37, 53, 16, 4, 3, 5, 16, 24, (2, 3), (1, 0, 2, 1)),      # six phases, three blocks of filters
    (8, 8, 1, 1, 2, 1, 1, 1, (1, 1), (0, 0, 0, 0)),           # two pairs for eight waves, 56 pixels
    (8, 8, 1, 1, 1, 2, 1, 9, (1, 1), (0, 0, 0, 1)),           # 64 pixels, one filter beyond a block
    (13, 5, 3, 1, 3, 3, 3, 7, (1, 1), (1, 1, 1, 1)),          # 65 pixels
    (5, 4, 6, 2, 5, 4, 3, 10, (3, 3), (2, 2, 1, 2)),          # two groups of five filters, nine phases of one or two taps
    (9, 7, 4, 3, 2, 2, 4, 8, (3, 1), (0, 1, 1, 0)),           # a phase without taps: dzdx elsewhere
    (6, 7, 12, 2, 6, 2, 12, 20, (1, 2), (3, 2, 0, 1)),        # six filter rows: dzdw elsewhere
    (16, 16, 40, 4, 4, 4, 40, 24, (1, 1), (1, 2, 2, 1)),      # 640 pairs, 1024 pixels of dzdw
    (16, 17, 8, 4, 3, 3, 8, 16, (1, 1), (1, 1, 1, 1)),        # 1088: blocks of 1024
    (32, 32, 8, 4, 5, 5, 8, 16, (1, 1), (2, 2, 2, 2)),        # 4096 pixels, 13e6 products
    (33, 32, 8, 4, 5, 5, 8, 16, (1, 1), (2, 2, 2, 2)),        # 4224: the tile kernels
    (12, 11, 33, 3, 3, 3, 33, 30, (1, 1), (1, 1, 1, 1)),      # ragged channels and filters
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("precision", [B.MCN_PREC_FP32, B.MCN_PREC_FP32_PLAIN])
def test_every_element(case, precision):
    L = layer(*CASES[case], idx=case)
    e = U.run_layer_full(L, precision=precision, with_bias=bool(case % 2), seed=case, misalign=case % 2)
    # a sum of n terms rounds n times at most (and the bias once): n * 2^-24 of the sum of absolute values
    ho, wo = oracle.output_size(synth.x_shape(L), synth.w_shape(L), L["stride"], L["pad"])
    taps = L["Hf"] * L["Wf"]
    terms = {"forward": taps * L["Df"] + 1, "backward_data": taps * L["K"], "backward_filter": ho * wo * L["N"], "backward_bias": ho * wo * L["N"]}
    print("small layer", case, e, flush=True)
    for k, n in terms.items():
        assert e[k] <= max(n, 2) * 2.0 ** -24, (case, k, e[k], n)


@pytest.mark.parametrize("case", [0, 4, 7, 8])
def test_relu_and_both_derivatives_in_one_call(case):
    L = layer(*CASES[case], idx=case)
    st, pad = L["stride"], L["pad"]
    x, w, b = synth.make_x(L).cuda(), synth.make_w(L).cuda(), synth.make_b(L).cuda()
    y = B.conv_forward(x, w, b, st, pad)
    assert torch.equal(B.conv_relu_forward(x, w, b, st, pad), y.clamp(min=0.0))
    dz = synth.make_dzdy(L, y.shape[3], y.shape[2]).cuda()
    dw, db = B.conv_backward_filter_bias(x, w.shape, dz, st, pad)
    assert torch.equal(dw, B.conv_backward_filter(x, w.shape, dz, st, pad))
    assert torch.equal(db, B.conv_backward_bias(x.shape, w.shape, dz, st, pad))


def test_padding_meets_nothing():
    """Infinite weights and derivatives meet the samples that there are, and no zero in the place of one that there is not."""
    L = layer(9, 8, 5, 2, 3, 4, 5, 11, (1, 2), (1, 1, 2, 1), idx=50)
    st, pad = L["stride"], L["pad"]
    x, w = synth.make_x(L).abs() + 1.0, synth.make_w(L)
    w[:, 1, 0, 0], w[3, 2, 3, 2] = float("inf"), float("-inf")
    ref = torch.nn.functional.conv2d(torch.nn.functional.pad(x, (pad[0], pad[1], pad[2], pad[3]), value=0.0), torch.nan_to_num(w, 0.0, 0.0, 0.0), stride=(st[1], st[0]))
    # which windows meet the infinite taps inside the plane
    inside = torch.nn.functional.pad(torch.ones_like(x), (pad[0], pad[1], pad[2], pad[3]))
    hits = torch.nn.functional.conv2d(inside, torch.isinf(w).float(), stride=(st[1], st[0])) > 0
    y = B.conv_forward(x.cuda(), w.cuda(), None, st, pad).cpu()
    assert torch.equal(~torch.isfinite(y), hits) and not bool(hits.all())
    assert float((y - ref)[~hits].abs().max()) <= 1e-4
    dz = synth.make_dzdy(L, y.shape[3], y.shape[2])
    dz[1, 4, 0, 0] = float("inf")               # the corner: two of its columns and a row are padding
    dw = B.conv_backward_filter(x.cuda(), w.shape, dz.cuda(), st, pad).cpu()
    want = torch.zeros_like(dw, dtype=torch.bool)
    want[4, :, 2:, 1:] = True
    assert torch.equal(torch.isinf(dw), want) and not bool(torch.isnan(dw).any())
    dx = B.conv_backward_data(x.shape, torch.nan_to_num(w, 0.0, 0.0, 0.0).cuda(), synth.make_dzdy(L, y.shape[3], y.shape[2]).cuda(), st, pad)
    assert bool(torch.isfinite(dx).all())


def test_replays_of_a_graph():
    L = layer(*CASES[0], idx=60)
    st, pad = L["stride"], L["pad"]
    x, w, b = synth.make_x(L).cuda(), synth.make_w(L).cuda(), synth.make_b(L).cuda()
    dz = torch.randn_like(B.conv_forward(x, w, b, st, pad))

    def passes():
        return [B.conv_forward(x, w, b, st, pad), *B.conv_backward_filter_bias(x, w.shape, dz, st, pad), B.conv_backward_data(x.shape, w, dz, st, pad)]
    eager = passes()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = passes()
    for _ in range(3):
        for t in captured:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, c) for a, c in zip(eager, captured))
