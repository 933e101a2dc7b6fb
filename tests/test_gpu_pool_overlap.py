"""Pooling forward and max pooling derivative with overlapping (or spaced) 2x2 and 3x3 windows, one pass: where blocks of several planes and strips
of columns begin and end.  A derivative is the sum of at most four values of dzdy: 4 * 2^-24 of the sum of their sizes."""
import pytest

import parity_util as U
from test_gpu_pool_parity import player, run_pool

pytestmark = pytest.mark.gpu

CASES = [  # H, W, D, N, window, stride, pad
    (1, 1, 3, 5, 2, (1, 1), (1, 1, 1, 1)),         # more windows than samples
    (13, 13, 7, 5, 3, (2, 2), (0, 1, 0, 1)),       # few planes: one per block
    (13, 11, 64, 50, 3, (2, 2), (0, 1, 0, 1)),     # several planes per block, the last block short
    (64, 64, 3, 2, 3, (2, 2), (0, 1, 0, 1)),       # one plane exactly fills a block
    (65, 64, 3, 2, 3, (2, 2), (1, 0, 0, 1)),       # the first size in strips
    (224, 37, 2, 2, 3, (2, 2), (0, 0, 2, 2)),      # strips of uneven width
    (300, 50, 2, 1, 2, (1, 1), (1, 0, 1, 0)),      # every sample in four windows
    (100, 90, 2, 1, 3, (2, 3), (0, 0, 0, 0)),      # unequal strides, columns past the last window
    (120, 61, 2, 1, 2, (3, 4), (0, 1, 1, 0)),      # spaced windows: samples in none, strips that begin between windows
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
