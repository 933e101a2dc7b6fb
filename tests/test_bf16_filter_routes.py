"""Layers whose filter derivative takes operands rounded to bf16 whatever their pads and sizes: vertical stride 1, filters of at most five rows, more than 32
filters a group.  Their route is asked for on the host; on the GPU the smaller ones are compared with the oracle."""
import pytest
import torch

import oracle
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth

import parity_util as U

BF = B.MCN_PREC_BF16

SMALL = [
    # H  W  D  N  Hf Wf Df K   stride  pad
    # pads above the plane that several patches of rows reach into
    (12, 6, 1, 5, 1, 2, 1, 220, (1, 1), (28, 25, 2, 0)),
    (23, 10, 90, 3, 3, 3, 90, 140, (1, 1), (40, 8, 1, 4)),
    (16, 27, 48, 2, 3, 3, 12, 140, (1, 1), (19, 3, 5, 0)),
    (2, 5, 96, 5, 3, 5, 48, 102, (1, 2), (32, 2, 0, 2)),
    (109, 19, 325, 2, 1, 1, 325, 39, (1, 1), (29, 6, 0, 0)),
    (44, 13, 5, 4, 1, 3, 5, 152, (1, 1), (28, 0, 1, 4)),
    # one column of at most four rows, one or two images: an odd number of octets
    (4, 2, 30, 1, 2, 2, 30, 158, (1, 1), (0, 0, 0, 0)),
    (3, 1, 212, 2, 3, 1, 53, 148, (1, 1), (0, 1, 0, 0)),
    (2, 2, 7, 1, 1, 1, 7, 374, (1, 1), (0, 0, 0, 0)),
    (1, 3, 4, 2, 1, 1, 1, 248, (1, 3), (0, 0, 0, 0)),
    (9, 3, 16, 1, 1, 2, 16, 65, (1, 2), (1, 2, 0, 0)),
    # the same where two columns of x are more than a unit holds
    (3, 74, 558, 2, 3, 2, 279, 76, (1, 11), (0, 0, 0, 0)),
    # one column of at most four rows of many images, two pairs of which are more than a unit holds
    (3, 2, 369, 87, 1, 6, 369, 38, (1, 9), (1, 0, 2, 3)),
]

# Images of more than 512 MiB, one and two pairs of which are too much for the offsets of a unit
LARGE = [
    (60, 2289, 6, 4, 3, 2, 6, 961, (1, 1), (4, 9, 9, 3)),
    (844, 485, 160, 5, 3, 1, 80, 654, (1, 1), (1, 3, 0, 0)),
    (691, 656, 848, 1, 1, 1, 212, 680, (1, 2), (3, 1, 0, 1)),
    (2935, 3813, 13, 2, 2, 7, 13, 35, (1, 1), (3, 3, 2, 3)),
    (1036, 3264, 76, 2, 3, 3, 38, 158, (1, 1), (3, 2, 3, 1)),
    (83410, 25, 234, 2, 2, 1, 234, 68, (1, 1), (0, 0, 0, 0)),
    (1387, 2399, 9, 1, 3, 2, 9, 101, (1, 1), (1, 1, 1, 1)),
    # of dzdy and of x; three of them: the last one has no other in its pair
    (701, 1103, 8, 3, 3, 1, 8, 450, (1, 1), (1, 1, 0, 0)),
    (823, 821, 403, 3, 2, 2, 403, 34, (1, 1), (2, 0, 0, 1)),
]


def _layer(case):
    H, W, D, N, Hf, Wf, Df, K, st, pad = case
    return dict(H=H, W=W, D=D, N=N, Hf=Hf, Wf=Wf, Df=Df, K=K, stride=st, pad=pad)


@pytest.mark.parametrize("case", SMALL + LARGE)
def test_route(case):
    L = _layer(case)
    d = B.make_desc((L["N"], L["D"], L["W"], L["H"]), (L["K"], L["Df"], L["Wf"], L["Hf"]), L["stride"], L["pad"], BF)
    assert B.mcn_conv_kernel_name(d, B.MCN_OP_BACKWARD_FILTER) == "wgrad_bf16" and B.mcn_conv_operand_planes(d, B.MCN_OP_BACKWARD_FILTER) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(SMALL)))
def test_small_layers(case):
    L = dict(_layer(SMALL[case]), config=8, index=300 + case)
    x, w = synth.make_x(L), synth.make_w(L)
    ho, wo = oracle.output_size(x.shape, w.shape, L["stride"], L["pad"])
    p = synth.make_dzdy(L, ho, wo)
    print("bf16 filter derivative", SMALL[case], flush=True)
    got = B.conv_backward_filter(x.cuda(), w.shape, p.cuda(), L["stride"], L["pad"], BF).cpu().numpy()
    xr, pr = (U.np64(t.to(torch.bfloat16).to(torch.float32)) for t in (x, p))
    ref = oracle.backward_filter(xr, w.shape, pr, L["stride"], L["pad"])
    den = oracle.backward_filter(abs(xr), w.shape, abs(pr), L["stride"], L["pad"])
    # sums of products that fp32 holds exactly: n * 2^-24 of the sum of absolute values at most, n < 2^13 products with a sample of the plane
    assert U.norm_err(got, ref, den) <= 2.0 ** -11


@pytest.mark.gpu
@pytest.mark.parametrize("case", LARGE[-2:])
def test_large_images(case):
    H, W, D, N, Hf, Wf, Df, K, st, pad = case
    g = torch.Generator(device="cuda").manual_seed(H)
    Ho, Wo = oracle.output_size((N, D, W, H), (K, Df, Wf, Hf), st, pad)
    # -1, 0 and 1: sums of some two million products are exact in fp32
    x, p = (torch.randint(-1, 2, s, device="cuda", generator=g).float() for s in ((N, D, W, H), (N, K, Wo, Ho)))
    print("bf16 filter derivative, large images", case, flush=True)
    got = B.conv_backward_filter(x, (K, Df, Wf, Hf), p, st, pad, BF)
    ref = torch.zeros_like(got)
    for n in range(N):
        for j in range(Wo):
            for fj in range(Wf):
                if not 0 <= j + fj - pad[2] < W:
                    continue
                for fi in range(Hf):
                    lo, hi = max(0, pad[0] - fi), min(Ho, H + pad[0] - fi)       # rows of dzdy that meet one of x
                    ref[:, :, fj, fi] += p[n, :, j, lo:hi].contiguous() @ x[n, :, j + fj - pad[2], lo + fi - pad[0]:hi + fi - pad[0]].contiguous().T
    assert torch.equal(got, ref)
