"""Pooling forward and max pooling derivative with overlapping (or spaced) 2x2 and 3x3 windows: where blocks of several planes and strips
of columns begin and end (which calls take the kernels that go through LDS: pool_derivative_in_lds, pool_forward_in_lds in
csrc/kern_pool.h, tests/pool_tiles_check.cpp).  A derivative is the sum of at most four values of dzdy: 4 * 2^-24 of the sum of their sizes."""
import pytest
import torch

from paper_1412_4564_amd import binding as B
from test_gpu_pool_parity import player, run_pool

pytestmark = pytest.mark.gpu

CASES = [  # H, W, D, N, window, stride, pad
    (1, 1, 3, 5, 2, (1, 1), (1, 1, 1, 1)),         # more windows than samples
    (13, 13, 7, 5, 3, (2, 2), (0, 1, 0, 1)),       # few planes: one per block
    (13, 11, 64, 50, 3, (2, 2), (0, 1, 0, 1)),     # several planes per block, the last block short
    (64, 64, 3, 2, 3, (2, 2), (0, 1, 0, 1)),       # few large blocks: the two-pass kernels
    (65, 64, 3, 2, 3, (2, 2), (1, 0, 0, 1)),
    (224, 37, 2, 2, 3, (2, 2), (0, 0, 2, 2)),
    (64, 64, 40, 8, 3, (2, 2), (0, 1, 0, 1)),      # enough blocks: one plane exactly fills a block
    (65, 64, 20, 8, 3, (2, 2), (1, 0, 0, 1)),      # the first size in strips
    (224, 37, 30, 4, 3, (2, 2), (0, 0, 2, 2)),     # strips of uneven width
    (300, 50, 8, 7, 3, (2, 2), (2, 1, 1, 0)),      # narrow strips, odd pads
    (300, 50, 2, 1, 2, (1, 1), (1, 0, 1, 0)),      # every sample in four windows
    (100, 90, 2, 1, 3, (2, 3), (0, 0, 0, 0)),      # unequal strides, columns past the last window
    (120, 61, 2, 1, 2, (3, 4), (0, 1, 1, 0)),      # spaced windows: samples in none
    (700, 9, 1, 2, 3, (2, 2), (0, 0, 0, 0)),       # too tall for strips: the two-pass kernels
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_average_forward_every_element(case):
    H, W, D, N, f, stride, pad = CASES[case]
    e = run_pool(player(H, W, D, N, (f, f), stride, pad, "avg", idx=80 + case), seed=case)
    assert e[0] <= 9 * 2.0 ** -24 + 2.0 ** -23, e      # nine additions and a division


@pytest.mark.parametrize("case", range(len(CASES)))
def test_derivative_every_element(case):
    H, W, D, N, f, stride, pad = CASES[case]
    e = run_pool(player(H, W, D, N, (f, f), stride, pad, "max", idx=60 + case), seed=case)
    assert e[1] <= 4 * 2.0 ** -24, e


LARGE = [  # beyond 128 MiB, where the forward pass goes through LDS: H, W, D, N, window, stride, pad
    (55, 57, 96, 115, 3, (2, 2), (0, 1, 0, 1)),    # one plane per block
    (13, 11, 512, 470, 3, (1, 2), (1, 1, 2, 0)),   # 28 planes per block, unequal strides
    (91, 93, 64, 63, 2, (1, 1), (1, 0, 0, 1)),     # strips of window columns
]


@pytest.mark.parametrize("method", ["max", "avg"])
@pytest.mark.parametrize("case", range(len(LARGE)))
def test_forward_of_large_inputs(case, method):
    H, W, D, N, f, stride, pad = LARGE[case]
    x = torch.randn(N, D, W, H, generator=torch.Generator(device="cuda").manual_seed(case), device="cuda")
    assert x.numel() >= 1 << 25
    y = B.pool_forward(x, (f, f), stride, pad, B.MCN_POOL_MAX if method == "max" else B.MCN_POOL_AVG)
    # torch's rows and columns are the second-last and the last axis: columns, then rows here
    xp = torch.nn.functional.pad(x, (pad[0], pad[1], pad[2], pad[3]), value=float("-inf") if method == "max" else 0.0)
    if method == "max":
        assert torch.equal(y, torch.nn.functional.max_pool2d(xp, f, (stride[1], stride[0])))
        return
    inside = torch.nn.functional.pad(torch.ones(1, 1, W, H, device="cuda"), (pad[0], pad[1], pad[2], pad[3]))
    ref, den, n = torch.zeros_like(y), torch.zeros_like(y), 0
    for j in range(f):
        for i in range(f):
            cols, rows = slice(j, j + (y.shape[2] - 1) * stride[1] + 1, stride[1]), slice(i, i + (y.shape[3] - 1) * stride[0] + 1, stride[0])
            ref += xp[:, :, cols, rows]; den += xp[:, :, cols, rows].abs(); n = n + inside[:, :, cols, rows]
    # both sums of at most nine numbers and a division in fp32
    assert float(((y - ref / n).abs() / (den / n)).max()) <= 2 * (9 * 2.0 ** -24 + 2.0 ** -23)
