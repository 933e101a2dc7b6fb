"""Input derivatives of strided layers whose phases are packed by one launch, and those that are not: every result against the oracle, with phases that
differ in taps and units, phases without taps, and a workspace of exactly the size that was asked for."""
import pytest
import torch

import oracle
from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth

import parity_util as U

pytestmark = pytest.mark.gpu

CASES = [
    # H  W  D  N  Hf Wf Df K   stride  pad
    (23, 20, 40, 2, 3, 3, 40, 70, (2, 2), (1, 0, 0, 1)),     # four phases of four, two, two and one taps
    (17, 30, 33, 3, 3, 5, 33, 20, (1, 2), (1, 1, 2, 2)),     # two phases
    (22, 25, 36, 2, 4, 7, 36, 35, (2, 3), (0, 1, 1, 2)),     # six phases
    (25, 26, 48, 2, 5, 4, 24, 66, (3, 3), (0, 0, 0, 0)),     # nine phases, two groups, of four to one taps
    (30, 27, 34, 1, 5, 4, 34, 40, (4, 3), (2, 1, 0, 0)),     # twelve phases: packed one by one
    (21, 22, 130, 2, 2, 2, 130, 129, (3, 3), (0, 0, 0, 0)),  # nine phases, five of them without taps
    (48, 48, 64, 8, 6, 6, 64, 256, (2, 2), (2, 2, 2, 2)),    # four large phases, tiles shared between blocks
    (26, 31, 17, 5, 1, 3, 17, 17, (1, 3), (0, 0, 1, 1)),     # one tap in each of three phases, one channel past 16
]
# fp32: n products are summed in fp32, n <= 256 * 9: far under the bar of the backward passes; bf16 operands are rounded to 2^-9 each, so a
# product is off by at most 2^-8, and two planes of each operand leave 2^-16 of it
BAR = {B.MCN_PREC_FP32: U.TOL_BWD / 10, B.MCN_PREC_BF16: 2.0 ** -8 * 1.05, B.MCN_PREC_FP32_BF16X3: 2.0 ** -14}


@pytest.mark.parametrize("precision", sorted(BAR))
@pytest.mark.parametrize("case", range(len(CASES)))
def test_phases_of_input_derivative(case, precision):
    H, W, D, N, Hf, Wf, Df, K, st, pad = CASES[case]
    L = dict(H=H, W=W, D=D, N=N, Hf=Hf, Wf=Wf, Df=Df, K=K, stride=st, pad=pad, config=9, index=900 + case)
    x, w = synth.make_x(L), synth.make_w(L)
    ho, wo = oracle.output_size(x.shape, w.shape, st, pad)
    p = synth.make_dzdy(L, ho, wo)
    d = B.make_desc(x.shape, w.shape, st, pad, precision)
    need = B.mcn_conv_workspace_size(d, 1)
    print("phases", CASES[case], precision, need, flush=True)
    wg, pg = w.cuda(), p.cuda()
    # a workspace of the size asked for and no more: what lies behind it stays as it was
    buf = torch.full((need // 4 + 1024,), 7.0, device="cuda")
    got = torch.full(tuple(x.shape), float("nan"), device="cuda")
    B.mcn_conv_backward_data(d, wg.data_ptr(), pg.data_ptr(), got.data_ptr(), buf.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.all(buf[need // 4:] == 7.0)
    ref = oracle.backward_data(x.shape, U.np64(w), U.np64(p), st, pad)
    den = oracle.backward_data(x.shape, abs(U.np64(w)), abs(U.np64(p)), st, pad)
    e = U.norm_err(got.cpu().numpy(), ref, den)
    assert e <= BAR[precision], e
