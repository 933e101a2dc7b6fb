"""Weights packed from runs of the caller's array (igemm_pack_runs_kernel, csrc/kern_igemm_split.h) on both sides of the size from which they are, against
sums in 64 bits: operands are whole numbers, which one, two or three planes hold exactly, and a weight in a wrong place or left out shows by its size."""
import pytest
import torch

from paper_1412_4564_amd import binding as B

pytestmark = pytest.mark.gpu

P3, P2, P1 = B.MCN_PREC_FP32, B.MCN_PREC_FP32_BF16X3, B.MCN_PREC_BF16
CASES = [  # H, W, N, Hf, Wf, channels of a group, filters, groups, precision
    (14, 14, 1, 3, 3, 512, 512, 1, P3),       # row pairs: forward by runs, dzdx not
    (14, 14, 1, 3, 3, 507, 500, 1, P3),       # ragged in both directions
    (14, 14, 8, 5, 5, 512, 256, 1, P3),
    (14, 13, 8, 3, 4, 500, 490, 1, P3),
    (14, 14, 8, 5, 5, 250, 131, 1, P3),       # too few blocks
    (7, 7, 4, 3, 3, 512, 512, 1, P2),
    (9, 8, 3, 5, 5, 250, 259, 1, P2),         # runs whose length no four divide
    (8, 7, 2, 2, 1, 741, 1501, 1, P2),        # two taps, the fewest
    (12, 11, 2, 4, 8, 250, 262, 1, P2),       # 32 taps, the most
    (12, 11, 2, 3, 11, 250, 262, 1, P2),      # 33
    (9, 9, 2, 3, 3, 256, 640, 2, P2),         # two groups
    (7, 7, 4, 3, 3, 512, 512, 1, P1),
    (9, 8, 3, 5, 5, 263, 250, 1, P1),
    (9, 9, 2, 7, 4, 130, 666, 2, P1),
    (7, 6, 3, 3, 3, 250, 131, 1, P1),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_forward_and_derivative(case):
    H, W, N, Hf, Wf, Df, K, G, precision = CASES[case]
    g = torch.Generator().manual_seed(case)
    pad = ((Hf - 1) // 2, Hf // 2, (Wf - 1) // 2, Wf // 2)
    most = {P1: 2 ** 7, P2: 2 ** 14, P3: 2 ** 17}[precision]

    def some(shape):                           # one in ten is not zero
        return torch.randint(-2, 3, shape, generator=g).float() * (torch.rand(shape, generator=g) < 0.125)
    x, dz = some((N, G * Df, W, H)), some((N, K, W, H))
    w = 2.0 * torch.randint(-most + 1, most, (K, Df, Wf, Hf), generator=g).float()       # even: row pairs halve sums of rows
    if case % 2:                               # weights that start at no multiple of 16 bytes
        store = torch.empty(w.numel() + 1, device="cuda")
        wg = store[1:].view(w.shape)
        wg.copy_(w)
    else:
        wg = w.cuda()
    print("weight runs", CASES[case], flush=True)
    y = B.conv_forward(x.cuda(), wg, None, (1, 1), pad, precision).cpu().double()
    dx = B.conv_backward_data(x.shape, wg, dz.cuda(), (1, 1), pad, precision).cpu().double()

    def forward(x, w):
        return torch.nn.functional.conv2d(torch.nn.functional.pad(x.double(), pad), w.double(), groups=G)

    def backward(w, dz):
        full = torch.nn.functional.conv_transpose2d(dz.double(), w.double(), groups=G)
        return full[:, :, pad[2]:pad[2] + W, pad[0]:pad[0] + H]
    # Products and the sums of each pair of planes are whole numbers below 2^24, so one and two planes round only where the two planes and the pieces of a
    # tile (32 at most) are put together: a rounding each, as do three planes
    for got, ref, size in ((y, forward(x, w), forward(x.abs(), w.abs())), (dx, backward(w, dz), backward(w.abs(), dz.abs()))):
        assert bool(((got - ref).abs() <= 40 * 2.0 ** -24 * size).all()), (CASES[case], float((got - ref).abs().max()))
