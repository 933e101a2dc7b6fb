"""The fp32 filter derivative on the bf16 matrix core with operands in three bf16 planes (kern_wgrad_split.h): every coefficient
against the oracle at the edges of tiles, patches, image pairs and the column ring, and the values that a split operand cannot carry."""
import numpy as np
import pytest
import torch

import oracle
import parity_util as U
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth
from test_gpu_parity import custom_layer

pytestmark = pytest.mark.gpu

# An MFMA rounds its running sum four times on the way through its 16 terms, each time by at most 2^-25 of it, and a running sum is at
# most the sum of |x||dzdy|: n terms are off by at most n/4 * 2^-25 of that, and with random signs by about sqrt(n/4) * 2^-25.  The
# largest n here is 40 * 40 * 24 = 38400: 2.9e-6; 1e-5 leaves a factor 3.
BOUND = 1e-5

CASES = [  # H, W, D, N, Hf, Wf, Df, K, stride, pad
    (27, 27, 96, 16, 5, 5, 48, 256, (1, 1), (2, 2, 2, 2)),       # two groups, seven quads to a column, the last of three rows
    (16, 16, 32, 100, 5, 5, 32, 32, (1, 1), (2, 2, 2, 2)),       # tiles of 32 filters
    (13, 19, 40, 41, 5, 3, 40, 72, (1, 1), (2, 0, 1, 2)),        # odd batch, filters ragged against 128, pads of one side
    (28, 30, 65, 9, 4, 4, 65, 130, (2, 2), (1, 1, 1, 1)),        # two row phases, one channel and two filters past a tile
    (61, 40, 7, 24, 7, 6, 7, 100, (3, 2), (3, 1, 0, 2)),         # three row phases, whole sweeps of few columns
    (96, 90, 3, 24, 11, 11, 3, 96, (4, 4), (0, 2, 0, 1)),        # four row phases, three channels
    (120, 121, 64, 24, 2, 2, 64, 80, (3, 3), (0, 0, 0, 0)),      # filter smaller than the stride: columns and rows that no window reads
    (28, 28, 160, 24, 1, 1, 160, 128, (1, 1), (0, 0, 0, 0)),     # 1x1: planes as columns
    (9, 7, 300, 77, 1, 1, 150, 260, (1, 1), (0, 0, 0, 0)),       # 1x1 in two groups, 63 rows, odd batch
    (30, 31, 200, 10, 1, 1, 200, 96, (2, 2), (0, 0, 0, 0)),      # 1x1 at stride 2
    (20, 24, 112, 32, 3, 5, 112, 200, (1, 1), (1, 1, 2, 2)),     # whole and shared tiles, chunks of few units
    (7, 8, 500, 12, 5, 5, 500, 520, (1, 1), (2, 2, 2, 2)),       # more tiles than compute units: tiles that one block computes
]


def planes(L, precision=B.MCN_PREC_FP32):
    return B.mcn_conv_operand_planes(B.make_desc(synth.x_shape(L), synth.w_shape(L), L["stride"], L["pad"], precision), B.MCN_OP_BACKWARD_FILTER)


def derivative(L, x, p, precision=B.MCN_PREC_FP32):
    dw = torch.full(synth.w_shape(L), -7.0, device="cuda")
    return B.conv_backward_filter(x, synth.w_shape(L), p, L["stride"], L["pad"], precision, out=dw)


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_every_coefficient(case, misalign):
    L = custom_layer(*CASES[case], idx=860 + case)
    st, pad = L["stride"], L["pad"]
    assert planes(L) == planes(L, B.MCN_PREC_FP32_BF16X3) == 3 and planes(L, B.MCN_PREC_FP32_PLAIN) == 0
    x, w = synth.make_x(L, case), synth.make_w(L, case)
    p = synth.make_dzdy(L, *oracle.output_size(x.shape, w.shape, st, pad), case)
    xd, pd = U.np64(x), U.np64(p)
    xg, pg = U.gpu(x, misalign), U.gpu(p, misalign)
    got = derivative(L, xg, pg)
    e = U.norm_err(got.cpu().numpy(), oracle.backward_filter(xd, w.shape, pd, st, pad), oracle.backward_filter(np.abs(xd), w.shape, np.abs(pd), st, pad))
    print("filter derivative in three planes", case, misalign, e, flush=True)
    assert e <= BOUND
    assert torch.equal(got, derivative(L, xg, pg)) and torch.equal(got, derivative(L, xg, pg, B.MCN_PREC_FP32_BF16X3))


# 1x1 filters at stride 1 whose windows run past the last row or column: those rows and columns of the output read nothing
@pytest.mark.parametrize("shape", [(28, 28, 160, 24, 128), (27, 14, 300, 33, 70), (9, 7, 300, 77, 260), (26, 25, 96, 24, 64)])
@pytest.mark.parametrize("pad", [(0, 1, 0, 0), (0, 2, 0, 1), (0, 0, 0, 1), (0, 5, 0, 2)])
def test_pointwise_with_pads_below_and_to_the_right(shape, pad):
    h, w_, d, n, k = shape
    L = custom_layer(h, w_, d, n, 1, 1, d, k, pad=pad, idx=870)
    assert planes(L) == 3
    x, w = synth.make_x(L, 4), synth.make_w(L, 4)
    p = synth.make_dzdy(L, h + pad[1], w_ + pad[3], 4)
    xd, pd = U.np64(x), U.np64(p)
    got = derivative(L, x.cuda(), p.cuda()).cpu().numpy()
    e = U.norm_err(got, oracle.backward_filter(xd, w.shape, pd, (1, 1), pad), oracle.backward_filter(np.abs(xd), w.shape, np.abs(pd), (1, 1), pad))
    print("pointwise filter derivative, pads", shape, pad, e, flush=True)
    assert e <= BOUND


@pytest.mark.parametrize("exponent", [-126, -118, -100, 0, 96])
def test_operands_of_every_size(exponent):
    """x scaled by a power of two: the planes hold it exactly, so the error stays that of ordinary operands (down to the rounding of
    subnormal products and results: half of 2^-149 for each of at most 25600 terms)."""
    L = custom_layer(*CASES[1], idx=880)
    x, w = synth.make_x(L, 1), synth.make_w(L, 1)
    p = synth.make_dzdy(L, 16, 16, 1)
    scaled = torch.ldexp(x, torch.tensor(exponent))
    xd, pd = U.np64(scaled), U.np64(p)
    got = derivative(L, scaled.cuda(), p.cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.backward_filter(xd, w.shape, pd, L["stride"], L["pad"])
    den = oracle.backward_filter(np.abs(xd), w.shape, np.abs(pd), L["stride"], L["pad"])
    worst = float(np.max(np.maximum(np.abs(got - ref) - 25600 * 2.0 ** -150 * 5, 0.0) / den))      # |dzdy| < 5
    print("filter derivative, x scaled by 2^%d: %.2e" % (exponent, worst), flush=True)
    assert worst <= BOUND


@pytest.mark.parametrize("case", [0, 3, 5, 7, 11])
def test_values_that_are_not_finite(case):
    """Coefficients that meet an infinity, a NaN or an overflow are those of the plain sum over the samples inside the array, all others
    as without them (up to the order of their sum: taps that meet such a value with a zero of the padding are summed again)."""
    L = custom_layer(*CASES[case], idx=890 + case)
    assert planes(L) == 3
    st, pad = L["stride"], L["pad"]
    x, w = synth.make_x(L, 2), synth.make_w(L, 2)
    p = synth.make_dzdy(L, *oracle.output_size(x.shape, w.shape, st, pad), 2)
    clean = derivative(L, x.cuda(), p.cuda()).cpu()
    n, d, wd, h = x.shape
    k, wo, ho = p.shape[1:]
    x[0, 0, wd // 2, h // 2], x[n - 1, d - 1, wd - 1, h // 2], p[n // 2, k - 1, wo - 1, 0] = float("inf"), 3.4e38, float("nan")
    got = derivative(L, x.cuda(), p.cuda()).cpu()
    # the coefficients that any of the three takes part in, and their sums
    mx, mp = torch.zeros_like(x), torch.zeros_like(p)
    mx[0, 0, wd // 2, h // 2] = mx[n - 1, d - 1, wd - 1, h // 2] = mp[n // 2, k - 1, wo - 1, 0] = 1.0
    one = lambda a, b: torch.from_numpy(oracle.backward_filter(U.np64(a), w.shape, U.np64(b), st, pad)).reshape(w.shape)
    touched = (one(mx, torch.ones_like(p)) + one(torch.ones_like(x), mp)) > 0
    assert touched.any() and not touched.all()
    den = one(torch.nan_to_num(x, posinf=0.0).abs().clamp(max=10.0), torch.nan_to_num(p).abs())
    assert ((got - clean).abs()[~touched] <= 2 * BOUND * den[~touched]).all()
    want = one(x, p)
    fits = want.abs() < 3.0e38
    assert torch.equal(torch.isnan(got[touched]), torch.isnan(want[touched]))
    inf = torch.isinf(want) & touched
    assert torch.equal(got[inf].double(), want[inf])
    ok = touched & fits & torch.isfinite(want)
    whole = one(torch.nan_to_num(x, posinf=0.0).abs(), torch.nan_to_num(p).abs())       # 3.4e38 among them
    assert ((got.double() - want).abs()[ok] <= BOUND * whole[ok]).all()


@pytest.mark.parametrize("case", [0, 1, 2, 3, 4, 5, 7, 8, 9, 11])
def test_coefficients_summed_again(case):
    """An operand that rounds to infinity in its first plane, where dzdy is tiny: every coefficient that it enters is summed again, to a
    result of ordinary size, in which no term may be missing or count twice."""
    L = custom_layer(*CASES[case], idx=910 + case)
    assert planes(L) == 3
    st, pad = L["stride"], L["pad"]
    x, w = synth.make_x(L, 5), synth.make_w(L, 5)
    p = synth.make_dzdy(L, *oracle.output_size(x.shape, w.shape, st, pad), 5)
    n, d, wd, h = x.shape
    mark = torch.zeros_like(x)
    mark[n - 1, d // 2, 0, h // 3] = mark[n // 2, 0, wd // 2, 0] = 1.0
    one = lambda a, b: torch.from_numpy(oracle.backward_filter(U.np64(a), w.shape, U.np64(b), st, pad)).reshape(w.shape)
    touched = one(mark, torch.ones_like(p)) > 0
    assert touched.any() and not touched.all()
    met = torch.from_numpy(oracle.forward(U.np64(mark), np.ones((L["K"], L["Df"], L["Wf"], L["Hf"])), None, st, pad)).reshape(p.shape) > 0
    x[mark > 0], p[met] = 3.4e38, 1e-37 * p[met]
    got, want, den = derivative(L, x.cuda(), p.cuda()).cpu().double(), one(x, p), one(x.abs(), p.abs())
    assert ((got - want).abs() <= BOUND * den).all()


# Fully-connected forward passes: the R terms of a result as two images of R/2, in the same kernel.  n = R here: below 3600.
FC_CASES = [  # H, W, D, N, K
    (4, 4, 96, 130, 1100),       # two images and 76 filters past a tile
    (1, 1, 282, 162, 2771),      # halves of 141 rows: the last quad holds one
    (7, 6, 61, 70, 900),         # halves of 1281 rows
    (3, 3, 394, 60, 1011),       # fewer than 64 images
]


@pytest.mark.parametrize("case", range(len(FC_CASES)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_fully_connected_forward(case, misalign):
    h, w_, d, n, k = FC_CASES[case]
    L = custom_layer(h, w_, d, n, h, w_, d, k, idx=900 + case)
    make = lambda precision: B.make_desc(synth.x_shape(L), synth.w_shape(L), L["stride"], L["pad"], precision)
    assert [B.mcn_conv_operand_planes(make(p), B.MCN_OP_FORWARD) for p in (B.MCN_PREC_FP32, B.MCN_PREC_BF16, B.MCN_PREC_FP32_PLAIN)] == [3, 3, 0]
    x, w, b = synth.make_x(L, case), synth.make_w(L, case), synth.make_b(L, case)
    xd, wd, bd = U.np64(x), U.np64(w), U.np64(b)
    xg, wg, bg = U.gpu(x, misalign), U.gpu(w, misalign), U.gpu(b, misalign)
    y = B.conv_forward(xg, wg, bg)
    e = U.norm_err(y.cpu().numpy(), oracle.forward(xd, wd, bd), oracle.forward(np.abs(xd), np.abs(wd), np.abs(bd)))
    print("fully-connected forward in three planes", case, misalign, e, flush=True)
    assert e <= BOUND
    assert torch.equal(y, B.conv_forward(xg, wg, bg, (1, 1), (0, 0, 0, 0), B.MCN_PREC_BF16))
    assert torch.equal(B.conv_relu_forward(xg, wg, bg), y.clamp(min=0.0))
    e0 = U.norm_err(B.conv_forward(xg, wg, None).cpu().numpy(), oracle.forward(xd, wd, None), oracle.forward(np.abs(xd), np.abs(wd), None))
    assert e0 <= BOUND
    # an infinity in the last term of an image, a NaN in the last weight of a filter: results that meet neither are as without them
    xg[n - 1, d - 1, w_ - 1, h - 1], wg[k - 2, d - 1, w_ - 1, h - 1] = float("inf"), float("nan")
    z = B.conv_forward(xg, wg, bg).reshape(n, k)
    assert torch.equal(z[:n - 1, :k - 2], y.reshape(n, k)[:n - 1, :k - 2]) and torch.isnan(z[:, k - 2]).all()
    others = [i for i in range(k) if i != k - 2]
    assert torch.equal(z[n - 1, others], torch.where(w[others, d - 1, w_ - 1, h - 1] > 0, float("inf"), float("-inf")).cuda())
