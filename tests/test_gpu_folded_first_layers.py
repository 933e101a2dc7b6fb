"""Strided layers of few channels whose forward pass folds the input's stride phases into channels (folded_view in csrc/igemm_plan.h, FOLDED in
csrc/kern_igemm_split.h): every result against 64-bit sums at unequal strides, all four pads, ragged phases, channels and filters, two groups; results
that are not finite are those of the plain sum."""
import pytest
import torch

from paper_1412_4564_amd import binding as B

pytestmark = pytest.mark.gpu

CASES = [  # H, W, D, N, Hf, Wf, Df, K, stride, pad
    (115, 117, 3, 48, 11, 11, 3, 96, (4, 4), (0, 0, 0, 0)),      # 48 channels of 3x3 taps
    (113, 110, 3, 48, 12, 10, 3, 70, (4, 4), (2, 3, 5, 1)),      # pads that are no multiple of the stride
    (100, 131, 2, 40, 9, 13, 2, 33, (3, 5), (4, 0, 1, 6)),       # unequal strides, 30 channels: the last group is not full
    (97, 90, 6, 40, 9, 9, 3, 80, (3, 3), (1, 2, 0, 3)),          # two groups of 40 filters
    (150, 140, 15, 8, 6, 3, 15, 24, (2, 1), (0, 1, 1, 1)),       # folded one way
]


def layer(case, seed=0):
    H, W, D, N, Hf, Wf, Df, K, st, pad = CASES[case]
    g = torch.Generator(device="cuda")
    g.manual_seed(2400 + 10 * case + seed)
    x = torch.randn((N, D, W, H), generator=g, device="cuda")
    w = torch.randn((K, Df, Wf, Hf), generator=g, device="cuda") * (2.0 / (Hf * Wf * Df)) ** 0.5
    b = torch.randn((K,), generator=g, device="cuda") * 0.1
    d = B.make_desc(x.shape, w.shape, st, pad)
    assert B.mcn_conv_operand_planes(d, B.MCN_OP_FORWARD) == 3 and B.mcn_conv_kernel_name(d, B.MCN_OP_FORWARD) == "igemm"
    return x, w, b, st, pad


def plain(x, w, b, st, pad):
    """In 64 bits, tap by tap."""
    N, D, W, H = x.shape
    K, Df, Wf, Hf = w.shape
    groups = D // Df
    xp = torch.nn.functional.pad(x.double(), pad)
    ho, wo = (H + pad[0] + pad[1] - Hf) // st[0] + 1, (W + pad[2] + pad[3] - Wf) // st[1] + 1
    y = torch.zeros((N, K, wo * ho), dtype=torch.float64, device=x.device)
    kg = K // groups
    for fj in range(Wf):
        for fi in range(Hf):
            v = xp[:, :, fj:fj + (wo - 1) * st[1] + 1:st[1], fi:fi + (ho - 1) * st[0] + 1:st[0]].reshape(N, D, wo * ho)
            for g in range(groups):
                y[:, g * kg:(g + 1) * kg] += torch.matmul(w[g * kg:(g + 1) * kg, :, fj, fi].double().contiguous(), v[:, g * Df:(g + 1) * Df].contiguous())
    return (y + b.double()[:, None]).reshape(N, K, wo, ho)


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("misalign", [0, 1])
def test_every_result(case, misalign):
    x, w, b, st, pad = layer(case)
    if misalign:
        x = torch.cat([x.new_zeros(misalign), x.reshape(-1)])[misalign:].reshape(x.shape)
    y = B.conv_forward(x, w, b, st, pad)
    den = plain(x.abs(), w.abs(), b.abs(), st, pad)
    e = float(((y.double() - plain(x, w, b, st, pad)).abs() / den).max())
    print("folded", case, misalign, e, flush=True)
    # n terms in planes that hold the operands exactly, rounded four times every sixteen elements: n / 4 * 2^-24, and the bias and the scales' sums
    n = w.shape[1] * w.shape[2] * w.shape[3]
    assert e <= (n / 4 + 4) * 2.0 ** -24
    assert torch.equal(y, B.conv_forward(x, w, b, st, pad)) and torch.equal(B.conv_relu_forward(x, w, b, st, pad), y.clamp(min=0.0))


@pytest.mark.parametrize("case", [0, 2, 3])
def test_values_that_are_not_finite(case):
    x, w, b, st, pad = layer(case, 1)
    clean = B.conv_forward(x, w, b, st, pad)
    x[0, 0, 20, 30], x[1, -1, 0, 0], x[2, 0, 41, 7] = float("inf"), float("nan"), float("-inf")
    w[3, 0, 0, 0], w[-1, -1, -1, -1] = float("inf"), 3.3e38
    y, ref = B.conv_forward(x, w, b, st, pad), plain(x, w, b, st, pad)
    # padding meets no tap: zeros there would make NaN of the infinite weight's products
    inside = torch.ones_like(x)
    met = plain(inside, torch.isinf(w).float(), torch.zeros_like(b), st, pad) > 0
    odd = ~torch.isfinite(ref)
    odd[:, 3] = met[:, 3] | odd[:, 3] & torch.isnan(ref[:, 3]) & met[:, 3]
    touched = plain((~torch.isfinite(x)).float(), torch.ones_like(w), torch.zeros_like(b), st, pad) > 0
    touched[:, 3] = True
    touched[:, -1] = True
    assert torch.equal(y[~touched], clean[~touched])
    assert not bool(torch.isfinite(y[:, 3])[met[:, 3]].any())
    others = [k for k in range(w.shape[0]) if k not in (3, w.shape[0] - 1)]
    assert torch.equal(torch.isnan(y[:, others]), torch.isnan(ref[:, others]))
    inf = torch.isinf(ref[:, others])
    assert bool(inf.any()) and torch.equal(y[:, others][inf].double(), ref[:, others][inf])
