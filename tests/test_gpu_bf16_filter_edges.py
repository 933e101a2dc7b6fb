"""Filter derivative with bf16 operands at the edges of its kernel's tiles, units and quads: sums over operands rounded beforehand, every
coefficient against the oracle at the fp32 bar, and inputs that are not finite."""
import numpy as np
import pytest
import torch

import oracle
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth

import parity_util as U

pytestmark = pytest.mark.gpu
BF = B.MCN_PREC_BF16

EDGES = [
    # H  W  D  N  Hf Wf Df K   stride  pad
    (5, 6, 33, 1, 1, 1, 33, 65, (1, 1), (0, 0, 0, 0)),       # one image: half of every pair is missing; planes as one column
    (28, 28, 130, 3, 1, 1, 130, 128, (1, 1), (0, 0, 0, 0)),  # 1x1, last pair half empty, filters fill the tile
    (9, 7, 40, 2, 1, 1, 40, 70, (1, 1), (2, 3, 1, 0)),       # 1x1 with pads on every side: rows above and below the plane
    (9, 7, 40, 2, 1, 1, 40, 70, (1, 1), (0, 3, 0, 0)),       # 1x1, more output rows than input rows
    (56, 4, 48, 2, 3, 3, 48, 64, (1, 1), (1, 1, 1, 1)),      # whole columns of 14 quads, fewer columns than filter and ring
    (57, 9, 86, 3, 3, 3, 86, 64, (1, 1), (1, 1, 1, 1)),      # 774 coefficients: a second tile of six; 57 rows: a quad of one row
    (31, 11, 43, 4, 3, 3, 43, 129, (1, 1), (1, 1, 1, 1)),    # 387 coefficients, 129 filters: remainders of both
    (14, 3, 30, 5, 3, 3, 30, 40, (1, 1), (4, 5, 3, 6)),      # pads above a quad: two lead quads, columns wholly outside
    (13, 13, 24, 33, 5, 5, 24, 48, (1, 1), (2, 2, 2, 2)),    # many images, odd
    (130, 5, 20, 2, 2, 4, 20, 36, (1, 3), (0, 1, 2, 0)),     # more rows than a patch holds, stride across wider than a unit's columns
    (6, 40, 34, 2, 4, 1, 17, 68, (1, 2), (3, 0, 0, 1)),      # two groups, one filter column: units share no column
]


@pytest.mark.parametrize("case", range(len(EDGES)))
def test_bf16_filter_derivative_edges(case):
    H, W, D, N, Hf, Wf, Df, K, st, pad = EDGES[case]
    L = dict(H=H, W=W, D=D, N=N, Hf=Hf, Wf=Wf, Df=Df, K=K, stride=st, pad=pad, config=8, index=case)
    x, w = synth.make_x(L), synth.make_w(L)
    ho, wo = oracle.output_size(x.shape, w.shape, st, pad)
    p = synth.make_dzdy(L, ho, wo)
    d = B.make_desc(x.shape, w.shape, st, pad, BF)
    assert B.mcn_conv_kernel_name(d, 2) == "wgrad_bf16" and B.mcn_conv_operand_planes(d, 2) == 1
    print("bf16 filter derivative", EDGES[case], flush=True)
    got = B.conv_backward_filter(x.cuda(), w.shape, p.cuda(), st, pad, BF).cpu().numpy()
    xr, pr = (U.np64(t.to(torch.bfloat16).to(torch.float32)) for t in (x, p))
    ref, den = oracle.backward_filter(xr, w.shape, pr, st, pad), oracle.backward_filter(abs(xr), w.shape, abs(pr), st, pad)
    # sums of products that fp32 holds exactly: n * 2^-24 of the sum of absolute values at most, n = N * Ho * Wo < 2^13
    assert U.norm_err(got, ref, den) <= 2.0 ** -11, U.norm_err(got, ref, den)


# The case and where the bad value is: the last sample of x's last plane or of dzdy's; or, in planes of 30 samples (7 quads and a half), the first of
# a channel, which the last quad of the plane before it holds beside rows of dzdy that are not there
BAD = [(c, where) for c in (1, 4, 6, 7, 9) for where in ("x", "dzdy")] + [(0, "x"), (0, "dzdy"), (0, "next channel")]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("case,where", BAD)
def test_bf16_filter_derivative_not_finite(case, where, bad):
    """One input that is not finite: the coefficients that meet it, and no other, are not finite, and which of the three they are."""
    H, W, D, N, Hf, Wf, Df, K, st, pad = EDGES[case]
    L = dict(H=H, W=W, D=D, N=N, Hf=Hf, Wf=Wf, Df=Df, K=K, stride=st, pad=pad, config=8, index=case)
    x, w = synth.make_x(L), synth.make_w(L)
    ho, wo = oracle.output_size(x.shape, w.shape, st, pad)
    p = synth.make_dzdy(L, ho, wo)
    if where == "dzdy":
        p[N - 1, K // 2, wo - 1, ho - 1] = bad
    elif where == "x":
        x[N - 1, D // 2, W - 1, H - 1] = bad
    else:
        x[N - 1, D // 2, 0, 0] = bad
    print("bf16 filter derivative, not finite", EDGES[case], where, bad, flush=True)
    got = B.conv_backward_filter(x.cuda(), w.shape, p.cuda(), st, pad, BF).cpu().numpy()
    xr, pr = (U.np64(t.to(torch.bfloat16).to(torch.float32)) for t in (x, p))
    with np.errstate(invalid="ignore"):
        ref = oracle.backward_filter(xr, w.shape, pr, st, pad)
    assert not np.all(np.isfinite(ref)) or case == 7        # padded so that no tap may meet the last sample
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin) and np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    # finite ones as above, or, formed again from the operands as they are, off by two roundings of 2^-9 each in every product
    xr[~np.isfinite(xr)] = 0; pr[~np.isfinite(pr)] = 0
    den = oracle.backward_filter(abs(xr), w.shape, abs(pr), st, pad)
    assert U.norm_err(got[fin], ref[fin], den[fin]) <= 2.0 ** -7.9
