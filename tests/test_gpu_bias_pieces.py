"""Bias derivative and its fused ReLU mask at the edges of their pieces and of the rule for one block a filter: planes around a row of loads, a piece
and the smallest plane of these kernels, arrays that do not begin at 16 bytes."""
import numpy as np
import pytest
import torch

from paper_1412_4564_amd import binding as B

import parity_util as U

pytestmark = pytest.mark.gpu

CASES = [  # plane, filters, images: pieces of 256 samples, one block a filter up to 48 of them
    ((8, 8), 5, 3), ((13, 5), 7, 48), ((13, 5), 7, 49), ((67, 1), 3, 2), ((17, 15), 4, 5), ((16, 16), 3, 48), ((257, 1), 3, 24), ((1, 257), 3, 25),
    ((31, 33), 2, 9), ((1, 511), 1, 1), ((64, 192), 1, 1), ((113, 109), 1, 1), ((100, 41), 300, 2),
]


@pytest.mark.parametrize("misalign", range(4))
@pytest.mark.parametrize("case", range(len(CASES)))
def test_bias_pieces(case, misalign):
    (wo, ho), K, N = CASES[case]
    rng = np.random.default_rng(case)
    # whole numbers: every sum is exact, so that a sample left out or counted twice shows whatever the number of the others
    p = torch.from_numpy((rng.integers(1, 9, (N, K, wo, ho)) * rng.choice((-1, 1), (N, K, wo, ho))).astype(np.float32))
    y = torch.from_numpy(np.maximum(rng.standard_normal((N, K, wo, ho), dtype=np.float32), 0))
    xs, ws = (N, 2, wo, ho), (K, 2, 1, 1)
    print("bias pieces", CASES[case], misalign, flush=True)
    pg, yg = U.gpu(p, misalign), U.gpu(y, (misalign + case) % 4)
    masked = U.np64(p) * (U.np64(y) > 0)
    assert np.array_equal(B.conv_backward_bias(xs, ws, pg).cpu().numpy(), U.np64(p).sum((0, 2, 3)))
    dzdp, dzdb = B.conv_relu_backward_bias(xs, ws, yg, pg)
    assert np.array_equal(dzdp.cpu().numpy(), masked) and np.array_equal(dzdb.cpu().numpy(), masked.sum((0, 2, 3)))
    dzdp, dzdb = B.conv_relu_backward_bias(xs, ws, yg, pg, inplace=True)
    assert dzdp.data_ptr() == pg.data_ptr() and np.array_equal(dzdp.cpu().numpy(), masked)
    assert np.array_equal(dzdb.cpu().numpy(), masked.sum((0, 2, 3)))
