"""1x1 layers whose pixels the three-plane kernel brings by fours (csrc/kern_igemm_split.h, QUADS): every result against the oracle where a four could
go wrong (planes of one four, the last one of the batch, tiles and groups of channels that are not full, arrays off 16-byte boundaries), and next to
layers whose planes are not whole fours."""
import pytest

import parity_util as U
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # H, W, D, N, Df, K, pad
    (2, 2, 144, 301, 144, 96, (0, 0, 0, 0)),      # an image is one four; the last tile is not full
    (4, 1, 160, 257, 160, 130, (0, 0, 0, 0)),     # ragged filters
    (1, 4, 131, 400, 131, 88, (0, 0, 0, 0)),      # channels odd against octets and units
    (12, 7, 200, 33, 100, 120, (0, 0, 0, 0)),     # two groups, 84 samples: an image ends inside a tile
    (30, 30, 40, 9, 40, 70, (0, 0, 0, 0)),        # units of fewer channel groups than fit
    (10, 10, 256, 30, 256, 48, (0, 0, 0, 0)),     # dzdx of 256 channels, forward in tiles of 64 filters
    (9, 9, 160, 40, 160, 96, (0, 0, 0, 0)),       # planes of 81: sample by sample
    (10, 10, 160, 30, 160, 96, (0, 0, 0, 0)),
    (10, 10, 160, 30, 160, 96, (0, 2, 0, 0)),     # the same plane, with rows that read nothing: sample by sample
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("misalign", [0, 1, 2])
def test_every_result(case, misalign):
    H, W, D, N, Df, K, pad = CASES[case]
    L = dict(H=H, W=W, D=D, N=N, Hf=1, Wf=1, Df=Df, K=K, stride=(1, 1), pad=pad, config=24, index=case)
    d = B.make_desc(synth.x_shape(L), synth.w_shape(L), (1, 1), pad)
    planes = [B.mcn_conv_operand_planes(d, op) for op in (B.MCN_OP_FORWARD, B.MCN_OP_BACKWARD_DATA)]
    assert 3 in planes
    e = U.run_layer_full(L, with_bias=bool(case % 2), seed=case, misalign=misalign)
    print("pointwise by fours", case, misalign, planes, e, flush=True)
    # sums of n terms, each rounded four times on the way through sixteen elements of the matrix core: n / 4 * 2^-24 of the sum of absolute values
    # for each of the three scales, of which the largest counts, and as much again for the pieces of a shared tile
    for name, terms in (("forward", Df + 1), ("backward_data", K)):
        assert e[name] <= max(terms, 16) / 2 * 2.0 ** -24, (case, name, e[name])
