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

# An MFMA rounds its running sum four times on the way through its 16 elements, each time by at most 2^-25 of it, and a running sum is
# at most the sum of |w||x|: n products are off by at most n/4 * 2^-25 of that, and with random signs by about sqrt(n/4) * 2^-25.  The
# largest n here is 128 * 25 = 3200 (dzdx of the two groups): 8.4e-7; 3e-6 leaves a factor 3.5 (measured: 1.3e-7).
BOUND = 3e-6


def planes(L, op):
    """3 where the pass (0 forward, 1 dzdx) takes the three-plane kernel."""
    return B.mcn_conv_operand_planes(B.make_desc(synth.x_shape(L), synth.w_shape(L), L["stride"], L["pad"]), op)


CASES = [  # H, W, D, N, Hf, Wf, Df, K, stride, pad, planes of forward and dzdx
    (40, 41, 16, 12, 5, 5, 16, 64, (1, 1), (2, 2, 2, 2), (3, 0)),      # one unit per tile, tile of 64 filters
    (11, 14, 40, 48, 5, 3, 40, 72, (1, 1), (2, 0, 1, 2), (3, 3)),      # channels ragged against 16, filters against 128
    (9, 10, 17, 46, 2, 2, 17, 33, (1, 1), (0, 1, 1, 0), (3, 3)),       # one channel and one filter past a unit and a tile
    (13, 12, 48, 37, 1, 2, 48, 130, (1, 1), (0, 0, 0, 0), (3, 3)),     # two taps
    (40, 36, 64, 16, 3, 3, 32, 80, (2, 1), (1, 1, 1, 1), (0, 3)),      # two groups of 40 filters, vertical stride: phases of dzdx
    (30, 30, 128, 16, 4, 4, 128, 200, (2, 2), (1, 1, 1, 1), (3, 3)),   # four phases, tiles shared between blocks
    (27, 27, 96, 8, 5, 5, 48, 256, (1, 1), (2, 2, 2, 2), (3, 3)),      # two groups, 25 taps; dzdx shared, tile of 64 filters
    (14, 14, 64, 16, 7, 7, 64, 72, (1, 1), (3, 3, 3, 3), (3, 0)),      # 49 taps, filter half as large as the plane
    (47, 39, 3, 80, 11, 11, 3, 64, (4, 4), (0, 0, 0, 0), (0, 3)),      # dzdx: 16 phases merged into 48 filters, rows that no window reads
    (52, 47, 4, 40, 5, 5, 4, 40, (2, 2), (2, 1, 0, 2), (0, 3)),        # dzdx: four phases of four channels, phases without a last row
    (95, 99, 6, 96, 4, 3, 3, 36, (3, 2), (1, 0, 2, 1), (0, 3)),        # dzdx: two groups of six phases
    (40, 40, 32, 16, 5, 5, 32, 70, (1, 1), (2, 2, 2, 2), (3, 3)),      # whole tiles of 128 x 128; dzdx 32 filters wide, shared
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_every_element(case, misalign):
    H, W, D, N, Hf, Wf, Df, K, st, pad, expect = CASES[case]
    L = custom_layer(H, W, D, N, Hf, Wf, Df, K, st, pad, idx=800 + case)
    assert (planes(L, 0), planes(L, 1)) == expect
    e = U.run_layer_full(L, with_bias=bool(case % 2), seed=case, misalign=misalign)
    U.assert_errors(e, label="three planes %d" % case)
    print("three planes, case", case, e, flush=True)
    assert e["forward"] <= BOUND and e["backward_data"] <= BOUND, e


PAIRS = [  # H, W, D, N, Df, K, pad: 3x3 layers both of whose passes take the kernel in row pairs, every tile in pieces
    (14, 14, 256, 2, 256, 256, (1, 1, 1, 1)),      # even plane
    (13, 9, 263, 3, 263, 260, (1, 1, 1, 1)),       # odd plane, ragged channels and filters
    (7, 16, 512, 1, 256, 516, (1, 0, 2, 1)),       # two groups of 258 filters, uneven pads
    (30, 5, 272, 1, 272, 288, (0, 0, 0, 0)),       # no pads; a third tile of 32 filters
]


@pytest.mark.parametrize("case", range(len(PAIRS)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_row_pairs_every_element(case, misalign):
    H, W, D, N, Df, K, pad = PAIRS[case]
    L = custom_layer(H, W, D, N, 3, 3, Df, K, (1, 1), pad, idx=820 + case)
    d = B.make_desc(synth.x_shape(L), synth.w_shape(L), (1, 1), pad)
    assert [B.mcn_conv_kernel_name(d, op) for op in (0, 1)] == ["igemm_f23"] * 2 and planes(L, 0) == planes(L, 1) == 3
    e = U.run_layer_full(L, with_bias=bool(case % 2), seed=case, misalign=misalign)
    U.assert_errors(e, label="three planes, row pairs %d" % case)
    print("three planes, row pairs", case, e, flush=True)
    # the error is bounded by the sums over all pairings of rows, up to three times a result's own: n = 3 * 263 * 3
    assert e["forward"] <= 2 * BOUND and e["backward_data"] <= 2 * BOUND, e


WHOLE = [  # H, W, D, N, K: row pairs, every tile one block's own
    (24, 27, 256, 25, 168),       # even plane: both rows of a pair in one 8-byte store, or in two where y is not aligned to 8 bytes
    (15, 15, 256, 31, 512),       # odd plane: a pair without a second row
]


@pytest.mark.parametrize("case", range(len(WHOLE)))
def test_row_pairs_in_whole_tiles(case):
    """Bias, ReLU, and results that are not finite, where the kernel writes its tiles itself; y at two alignments."""
    H, W, D, N, K = WHOLE[case]
    L = custom_layer(H, W, D, N, 3, 3, D, K, (1, 1), (1, 1, 1, 1), idx=825 + case)
    d = B.make_desc(synth.x_shape(L), synth.w_shape(L), (1, 1), (1, 1, 1, 1))
    assert B.mcn_conv_kernel_name(d, 0) == "igemm_f23" and planes(L, 0) == 3
    # no partial tiles in the workspace: packed weights only, 3 columns x 3 planes x 2 octets x 128 filters x 16 bytes per unit
    assert B.mcn_conv_workspace_size(d, 0) == (K + 127) // 128 * 4 * ((D + 15) // 16) * 9 * 2 * 128 * 16
    x, w, b = synth.make_x(L), synth.make_w(L), synth.make_b(L)
    ref = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=1)
    den = torch.nn.functional.conv2d(x.double().abs(), w.double().abs(), b.double().abs(), padding=1)
    flat = torch.empty(ref.numel() + 1, device="cuda")
    xg, wg, bg = x.cuda(), w.cuda(), b.cuda()
    for skip in (0, 1):
        out = flat[skip:skip + ref.numel()].view(ref.shape)
        assert out.data_ptr() % 8 == 4 * skip
        for relu in (False, True):
            out.fill_(-7.0)
            y = (B.conv_relu_forward if relu else B.conv_forward)(xg, wg, bg, (1, 1), (1, 1, 1, 1), out=out).cpu().double()
            e = float(((y - (ref.clamp(min=0) if relu else ref)).abs() / den).max())
            print("row pairs, whole tiles", case, skip, relu, e, flush=True)
            assert e <= 2 * BOUND           # as in the other row-pair tests
    # one infinite and one NaN sample, and a filter without a finite bias: its results, and the windows around the samples
    x[0, 3, 4, 5], x[N - 1, 0, W - 1, H - 1], b[7] = float("inf"), float("nan"), float("-inf")
    ref = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=1)
    for relu in (False, True):
        want = torch.where(torch.isnan(ref), torch.zeros_like(ref), ref.clamp(min=0)) if relu else ref
        y = (B.conv_relu_forward if relu else B.conv_forward)(x.cuda(), wg, b.cuda(), (1, 1), (1, 1, 1, 1)).cpu().double()
        assert torch.equal(torch.isnan(y), torch.isnan(want)) and torch.equal(torch.isinf(y), torch.isinf(want))
        inf, ok = torch.isinf(want), torch.isfinite(want)
        assert int(inf.sum()) > 0 and torch.equal(y[inf], want[inf])
        assert float(((y - want)[ok].abs() / den[ok]).max()) <= 2 * BOUND


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("shape", [(12, 12, 40, 6, 72, 5), (40, 40, 32, 16, 70, 5),     # shared tiles; whole tiles
                                   (14, 13, 256, 2, 96, 3)])                            # row pairs
def test_values_that_are_not_finite_or_nearly_so(relu, shape):
    """An infinite operand gives +-inf (or NaN) where the plain sum does, one near the largest float stays finite."""
    H, W, D, N, K, f = shape
    P = f // 2
    L = custom_layer(H, W, D, N, f, f, D, K, (1, 1), (P, P, P, P), idx=830)
    assert planes(L, 0) == 3
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
@pytest.mark.parametrize("shape", [(12, 12, 40, 6, 72, 5), (40, 40, 32, 16, 70, 5), (14, 13, 256, 2, 96, 3)])      # as above
def test_weights_and_biases_that_are_not_finite(where, shape):
    """An infinite weight or bias reaches every result of its filter (no pads: each meets all of the filter) and no other."""
    H, W, D, N, K, f = shape
    L = custom_layer(H, W, D, N, f, f, D, K, (1, 1), (0, 0, 0, 0), idx=831)
    assert planes(L, 0) == 3
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
    assert B.mcn_conv_operand_planes(B.make_desc(x.shape, w.shape, (1, 1), (2, 2, 2, 2)), 0) == 3
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


@pytest.mark.parametrize("N", [5, 40])      # shared tiles; whole tiles
def test_infinite_derivative_in_merged_phases(N):
    """dzdx of a strided first layer: an infinite dzdy reaches the samples of its window and no others."""
    w, p = torch.randn(64, 3, 7, 7), torch.randn(N, 64, 30, 31)
    p[0, 5, 7, 8], p[N - 1, 60, 29, 3] = float("inf"), float("-inf")
    x_shape = (N, 3, 2 * 29 + 7, 2 * 30 + 7)
    ref = torch.nn.functional.conv_transpose2d(p.double(), w.double(), stride=2)
    assert ref.shape == x_shape and B.mcn_conv_operand_planes(B.make_desc(x_shape, w.shape, (2, 2)), 1) == 3
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
    L = custom_layer(14, 13, 64, 4, 5, 5, 64, 72, (1, 1), (2, 2, 2, 2), idx=840)
    assert planes(L, 0) == 3
    x, w = synth.make_x(L) * scale, synth.make_w(L)
    ref = torch.nn.functional.conv2d(x.double(), w.double(), padding=2)
    den = torch.nn.functional.conv2d(x.double().abs(), w.double().abs(), padding=2)
    y = B.conv_forward(x.cuda(), w.cuda(), None, (1, 1), (2, 2, 2, 2)).cpu().double()
    assert float(((y - ref).abs() / den).max()) <= BOUND


@pytest.mark.parametrize("sx,sw", [(1e-34, 1), (1e-36, 1), (1e-37, 1), (1, 1e-37), (1e-37, 1e30), (1e30, 1e-37)])
@pytest.mark.parametrize("shape", [(14, 13, 64, 4, 72, 5), (14, 14, 256, 2, 96, 3)])       # any filter; row pairs
def test_operands_down_to_the_smallest_normal_number(sx, sw, shape):
    """The planes are scaled (split_bf16x3): operands of every size are held exactly.  Unscaled the last plane of an operand of
    1e-36 loses its bits (error 1e-5)."""
    H, W, D, N, K, f = shape
    L = custom_layer(H, W, D, N, f, f, D, K, (1, 1), (f // 2,) * 4, idx=841)
    assert planes(L, 0) == 3
    x, w = synth.make_x(L) * sx, synth.make_w(L) * sw
    ref = torch.nn.functional.conv2d(x.double(), w.double(), padding=f // 2)
    den = torch.nn.functional.conv2d(x.double().abs(), w.double().abs(), padding=f // 2)
    y = B.conv_forward(x.cuda(), w.cuda(), None, (1, 1), (f // 2,) * 4).cpu().double()
    err = float(((y - ref).abs() / den).max())
    print("three planes, small operands:", shape, sx, sw, err, flush=True)
    assert err <= BOUND
