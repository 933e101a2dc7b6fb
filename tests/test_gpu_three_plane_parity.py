"""fp32 convolutions on the bf16 matrix core with operands in three bf16 planes (kern_igemm_split.h): every element
against the oracle at the edges of tiles, units and channel groups, and the values that a split operand cannot carry."""
import numpy as np
import pytest
import torch

import parity_util as U
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth
from test_gpu_parity import custom_layer

pytestmark = pytest.mark.gpu

# The sum of n products in fp32 is off by at most n * 2^-24 of the sum of |w||x|, and by about sqrt(n) of that with random
# signs; the largest n here is 16 * 25 = 400 channels x taps (6 MFMA roundings per 16 of them): 3e-6 leaves a factor 2 on
# the random-sign figure 20 * 2^-24 = 1.2e-6.
BOUND = 3e-6

CASES = [  # H, W, D, N, Hf, Wf, Df, K, stride, pad
    (12, 11, 16, 3, 5, 5, 16, 64, (1, 1), (2, 2, 2, 2)),      # one unit per tap range, tile of 64 filters
    (11, 14, 40, 3, 5, 3, 40, 72, (1, 1), (2, 0, 1, 2)),      # channels ragged against 16, filters against 128
    (9, 10, 17, 2, 2, 2, 17, 33, (1, 1), (0, 1, 1, 0)),       # one channel and one filter past a unit and a tile
    (13, 12, 48, 4, 1, 2, 48, 130, (1, 1), (0, 0, 0, 0)),     # two taps
    (20, 18, 64, 2, 3, 3, 32, 24, (2, 1), (1, 1, 1, 1)),      # two groups of 12 filters, vertical stride: phases of dzdx
    (30, 30, 128, 6, 4, 4, 128, 200, (2, 2), (1, 1, 1, 1)),   # four phases, tiles shared between blocks
    (27, 27, 96, 8, 5, 5, 48, 256, (1, 1), (2, 2, 2, 2)),     # two groups, 25 taps in several ranges
    (7, 7, 32, 1, 7, 7, 32, 40, (1, 1), (3, 3, 3, 3)),        # one image, filter as large as the plane
    (47, 39, 3, 5, 11, 11, 3, 64, (4, 4), (0, 0, 0, 0)),      # dzdx: 16 phases merged into 48 filters, rows that no window reads
    (20, 17, 4, 3, 5, 5, 4, 40, (2, 2), (2, 1, 0, 2)),        # dzdx: four phases of four channels, phases without a last row
    (31, 33, 6, 2, 4, 3, 3, 36, (3, 2), (1, 0, 2, 1)),        # dzdx: two groups of six phases
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_every_element(case, misalign):
    H, W, D, N, Hf, Wf, Df, K, st, pad = CASES[case]
    L = custom_layer(H, W, D, N, Hf, Wf, Df, K, st, pad, idx=800 + case)
    e = U.run_layer_full(L, with_bias=bool(case % 2), seed=case, misalign=misalign)
    U.assert_errors(e, label="three planes %d" % case)
    print("three planes, case", case, e, flush=True)
    assert e["forward"] <= BOUND and e["backward_data"] <= BOUND, e


PAIRS = [  # H, W, D, N, Df, K, pad: 3x3 layers whose row pairs take the kernel (at least 256 channels, few tiles)
    (14, 14, 256, 2, 256, 256, (1, 1, 1, 1)),      # even plane: both rows of a pair in one store
    (13, 9, 263, 3, 263, 130, (1, 1, 1, 1)),       # odd plane (a pair without a second row), ragged channels and filters
    (7, 16, 512, 1, 256, 264, (1, 0, 2, 1)),       # two groups of 132 filters, uneven pads
    (30, 5, 272, 1, 272, 96, (0, 0, 0, 0)),        # no pads; tile of 128 filters, 96 used
]


@pytest.mark.parametrize("case", range(len(PAIRS)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_row_pairs_every_element(case, misalign):
    H, W, D, N, Df, K, pad = PAIRS[case]
    L = custom_layer(H, W, D, N, 3, 3, Df, K, (1, 1), pad, idx=820 + case)
    assert B.mcn_conv_kernel_name(B.make_desc(synth.x_shape(L), synth.w_shape(L), (1, 1), pad), 0) == "igemm_f23"
    e = U.run_layer_full(L, with_bias=bool(case % 2), seed=case, misalign=misalign)
    U.assert_errors(e, label="three planes, row pairs %d" % case)
    print("three planes, row pairs", case, e, flush=True)
    # the error is bounded by the sums over all pairings of rows, up to three times a result's own: n = 3 * 263 * 3
    assert e["forward"] <= 2 * BOUND and e["backward_data"] <= 2 * BOUND, e


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("shape", [(9, 10, 20, 2, 48, 5), (40, 40, 32, 16, 70, 5),      # shared tiles; whole tiles
                                   (14, 13, 256, 2, 96, 3)])                            # row pairs
def test_values_that_are_not_finite_or_nearly_so(relu, shape):
    """An infinite operand gives +-inf (or NaN) where the plain sum does, one near the largest float stays finite."""
    H, W, D, N, K, f = shape
    P = f // 2
    L = custom_layer(H, W, D, N, f, f, D, K, (1, 1), (P, P, P, P), idx=830)
    x, w, b = synth.make_x(L), synth.make_w(L), synth.make_b(L)
    x[0, 3, 4, 5], x[1, 7, 2, 2], x[N - 1, 0, W - 1, H - 1], x[1, 1, 7, 7] = float("inf"), float("-inf"), float("nan"), 3.4e38
    w[:, 1] *= 1e-4
    ref = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=P)
    xg, wg, bg = x.cuda(), w.cuda(), b.cuda()
    y = (B.conv_relu_forward if relu else B.conv_forward)(xg, wg, bg, (1, 1), (P, P, P, P)).cpu()
    if relu:
        ref = torch.where(torch.isnan(ref), torch.zeros_like(ref), ref.clamp(min=0))       # fmax(NaN, 0) = 0, as in the other kernels
    assert torch.equal(torch.isnan(y), torch.isnan(ref)) and torch.equal(torch.isinf(y), torch.isinf(ref))
    inf = torch.isinf(ref)
    assert int(inf.sum()) > 0 and torch.equal(y[inf].double(), ref[inf])
    ok = torch.isfinite(ref)
    den = torch.nn.functional.conv2d(torch.nan_to_num(x, 0, 0, 0).double().abs(), w.double().abs(), b.double().abs(), padding=P)
    assert float(((y.double() - ref)[ok].abs() / den[ok]).max()) <= 1e-5


@pytest.mark.parametrize("where", ["weight", "bias"])
@pytest.mark.parametrize("shape", [(9, 10, 20, 2, 48, 5), (40, 40, 32, 16, 70, 5), (14, 13, 256, 2, 96, 3)])      # as above
def test_weights_and_biases_that_are_not_finite(where, shape):
    """An infinite weight or bias reaches every result of its filter (no pads: each meets all of the filter) and no other."""
    H, W, D, N, K, f = shape
    L = custom_layer(H, W, D, N, f, f, D, K, (1, 1), (0, 0, 0, 0), idx=831)
    x, w, b = synth.make_x(L), synth.make_w(L), synth.make_b(L)
    if where == "weight":
        w[3, 2, 1, 0], w[K - 1, D - 1, f - 1, f - 1], w[5, 0, 0, 0] = float("inf"), float("-inf"), float("nan")
    else:
        b[3], b[K - 1], b[5] = float("inf"), float("-inf"), float("nan")
    ref = torch.nn.functional.conv2d(x.double(), w.double(), b.double())
    y = B.conv_forward(x.cuda(), w.cuda(), b.cuda()).cpu()
    assert torch.equal(torch.isnan(y), torch.isnan(ref)) and torch.equal(torch.isinf(y), torch.isinf(ref))
    inf = torch.isinf(ref)
    assert int(inf.sum()) == 2 * N * ref.shape[2] * ref.shape[3] and torch.equal(y[inf].double(), ref[inf])


def test_results_that_are_not_finite_do_not_hold_up_the_call():
    """27x27x96, 5x5x48x256 in two groups, 128 images.  Measured: 3.8, 5.1 and 2.4 times an ordinary call; one result after another,
    each to the end of its sum, 15, 16 and 97 times.  Bounds between the two."""
    x, w = torch.randn(128, 96, 27, 27, device="cuda"), torch.randn(256, 48, 5, 5, device="cuda") * 0.03
    out = torch.empty(128, 256, 27, 27, device="cuda")

    def best():
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(); B.conv_forward(x, w, None, (1, 1), (2, 2, 2, 2), out=out); b.record(); b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    ordinary, got = best(), {}
    kept = float(x[0, 0, 3, 3])
    for name, bound in (("nan", 10), ("inf", 12)):
        x[0, 0, 3, 3] = float(name)
        got[name] = (best() / ordinary, bound)
    x[0, 0, 3, 3] = kept
    x.fill_(float("nan"))
    got["all nan"] = (best() / ordinary, 12)
    print("three planes, not finite:", got, flush=True)
    assert all(t <= bound for t, bound in got.values()), got


@pytest.mark.parametrize("N", [2, 40])      # shared tiles; whole tiles
def test_infinite_derivative_in_merged_phases(N):
    """dzdx of a strided first layer: an infinite dzdy reaches the samples of its window and no others."""
    w, p = torch.randn(64, 3, 7, 7), torch.randn(N, 64, 30, 31)
    p[0, 5, 7, 8], p[N - 1, 60, 29, 3] = float("inf"), float("-inf")
    x_shape = (N, 3, 2 * 29 + 7, 2 * 30 + 7)
    ref = torch.nn.functional.conv_transpose2d(p.double(), w.double(), stride=2)
    assert ref.shape == x_shape
    dx = B.conv_backward_data(x_shape, w.cuda(), p.cuda(), (2, 2), (0, 0, 0, 0)).cpu()
    assert torch.equal(torch.isnan(dx), torch.isnan(ref)) and torch.equal(torch.isinf(dx), torch.isinf(ref))
    inf = torch.isinf(ref)
    assert int(inf.sum()) == 2 * 3 * 49 and torch.equal(dx[inf].double(), ref[inf])
    den = torch.nn.functional.conv_transpose2d(torch.nan_to_num(p, 0, 0, 0).double().abs(), w.double().abs(), stride=2)
    ok = torch.isfinite(ref)
    assert float(((dx.double() - ref)[ok].abs() / den[ok].clamp(min=1e-30)).max()) <= 1e-5


@pytest.mark.parametrize("scale", [1e30, 1e-20, 1e-30])
def test_scales(scale):
    """Powers of the fp32 range that a plane of half the width would lose: the error does not depend on the scale."""
    L = custom_layer(14, 13, 32, 2, 5, 5, 32, 64, (1, 1), (2, 2, 2, 2), idx=840)
    x, w = synth.make_x(L) * scale, synth.make_w(L)
    ref = torch.nn.functional.conv2d(x.double(), w.double(), padding=2)
    den = torch.nn.functional.conv2d(x.double().abs(), w.double().abs(), padding=2)
    y = B.conv_forward(x.cuda(), w.cuda(), None, (1, 1), (2, 2, 2, 2)).cpu().double()
    assert float(((y - ref).abs() / den).max()) <= BOUND


@pytest.mark.parametrize("sx,sw", [(1e-34, 1), (1e-36, 1), (1e-37, 1), (1, 1e-37), (1e-37, 1e30), (1e30, 1e-37)])
@pytest.mark.parametrize("shape", [(14, 13, 32, 2, 64, 5), (14, 14, 256, 2, 96, 3)])       # any filter; row pairs
def test_operands_down_to_the_smallest_normal_number(sx, sw, shape):
    """The planes are scaled (split_bf16x3): operands of every size are held exactly.  Unscaled the last plane of an operand of
    1e-36 loses its bits (error 1e-5)."""
    H, W, D, N, K, f = shape
    L = custom_layer(H, W, D, N, f, f, D, K, (1, 1), (f // 2,) * 4, idx=841)
    x, w = synth.make_x(L) * sx, synth.make_w(L) * sw
    ref = torch.nn.functional.conv2d(x.double(), w.double(), padding=f // 2)
    den = torch.nn.functional.conv2d(x.double().abs(), w.double().abs(), padding=f // 2)
    y = B.conv_forward(x.cuda(), w.cuda(), None, (1, 1), (f // 2,) * 4).cpu().double()
    err = float(((y - ref).abs() / den).max())
    print("three planes, small operands:", shape, sx, sw, err, flush=True)
    assert err <= BOUND
