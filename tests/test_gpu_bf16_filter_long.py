"""Filter derivative with bf16 operands where more than 2 GiB of an array lie behind a block's first patch, which is not the first of its sweep."""
import pytest
import torch

import oracle
from paper_1412_4564_amd import binding as B

pytestmark = pytest.mark.gpu
BF = B.MCN_PREC_BF16

CASES = [
    # H  W  D  N  Hf Wf Df K   stride  pad
    (112, 112, 16, 400, 3, 3, 16, 128, (1, 1), (1, 1, 1, 1)),     # dzdy of 2.6 GB
    (100, 90, 130, 638, 2, 3, 130, 40, (1, 1), (1, 0, 1, 1)),     # x of 3.0 GB
    (120, 64, 160, 600, 1, 1, 160, 40, (1, 1), (0, 0, 0, 1)),     # x of 2.9 GB, 1x1 filters
]


def reference(x, wshape, p, pad):
    """A column of all images at a time."""
    K, Df, Wf, Hf = wshape
    H, W, Ho, Wo = x.shape[3], x.shape[2], p.shape[3], p.shape[2]
    ref = torch.zeros(wshape, device="cuda")
    column = lambda t: t.permute(1, 0, 2).contiguous()
    for j in range(Wo):
        pj = column(p[:, :, j])
        for fj in range(Wf):
            if not 0 <= j + fj - pad[2] < W:
                continue
            xj = column(x[:, :, j + fj - pad[2]])
            for fi in range(Hf):
                lo, hi = max(0, pad[0] - fi), min(Ho, H + pad[0] - fi)           # rows of dzdy that meet one of x
                ref[:, :, fj, fi] += pj[:, :, lo:hi].reshape(K, -1) @ xj[:, :, lo + fi - pad[0]:hi + fi - pad[0]].reshape(Df, -1).T
    return ref


@pytest.mark.parametrize("case", range(len(CASES)))
def test_more_than_2_gib(case):
    H, W, D, N, Hf, Wf, Df, K, st, pad = CASES[case]
    g = torch.Generator(device="cuda").manual_seed(case)
    ho, wo = oracle.output_size((N, D, W, H), (K, Df, Wf, Hf), st, pad)
    # -1, 0 and 1: sums of up to six million products are exact in fp32
    x, p = (torch.randint(-1, 2, s, device="cuda", generator=g).float() for s in ((N, D, W, H), (N, K, wo, ho)))
    print("bf16 filter derivative, long arrays", CASES[case], flush=True)
    assert torch.equal(B.conv_backward_filter(x, (K, Df, Wf, Hf), p, st, pad, BF), reference(x, (K, Df, Wf, Hf), p, pad))
