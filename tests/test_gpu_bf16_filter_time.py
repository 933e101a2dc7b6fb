"""Filter derivative with bf16 operands where a sample is infinite: the sums that meet it are infinite as the matrix core leaves them, and cost
nothing; only those that a zero in the place of a missing sample makes NaN are formed again."""
import pytest
import torch

from paper_1412_4564_amd import binding as B

pytestmark = pytest.mark.gpu

LAYERS = [  # x, filters, stride, pad: tiles shared by many blocks, chunks, whole planes as columns
    ((128, 96, 27, 27), (256, 48, 5, 5), (1, 1), (2, 2, 2, 2)),
    ((64, 512, 28, 28), (128, 512, 1, 1), (1, 1), (0, 0, 0, 0)),
    ((32, 256, 56, 56), (256, 256, 3, 3), (1, 1), (1, 1, 1, 1)),
]


@pytest.mark.parametrize("where", ["x", "dzdy"])
@pytest.mark.parametrize("case", range(len(LAYERS)))
def test_one_infinity(case, where):
    xs, wsh, stride, pad = LAYERS[case]
    x, ws = torch.randn(xs, device="cuda").abs_().add_(0.5), B.Workspace()
    K, Wo, Ho = wsh[0], xs[2] + 2 * pad[2] - wsh[2] + 1, xs[3] + 2 * pad[0] - wsh[3] + 1
    p = torch.randn((xs[0], K, Wo, Ho), device="cuda").abs_().add_(0.5)
    out = torch.empty(wsh, device="cuda")

    def best():
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(); B.conv_backward_filter(x, wsh, p, stride, pad, B.MCN_PREC_BF16, out=out, workspace=ws); b.record(); b.synchronize()
            t.append(a.elapsed_time(b) * 1e3)
        return min(t)
    finite = best()
    # in the middle of a plane: no tap of it lies in the padding
    c, k, i = xs[1] // 3, K // 3, xs[3] // 2
    if where == "x":
        x[xs[0] // 2, c, xs[2] // 2, i] = -float("inf")
    else:
        p[xs[0] // 2, k, Wo // 2, Ho // 2] = -float("inf")
    inf = best()
    print("bf16 filter derivative, finite and with an infinity in %s: %.0f %.0f us" % (where, finite, inf), flush=True)
    # all of x and dzdy else is positive: -inf where a product with it is met, positive sums elsewhere
    Df, G = wsh[1], xs[1] // wsh[1]
    met = torch.zeros(wsh, dtype=torch.bool, device="cuda")
    if where == "x":
        met[c // Df * (K // G):(c // Df + 1) * (K // G), c % Df] = True
    else:
        met[k] = True
    assert torch.equal(out == -float("inf"), met) and torch.all(out[~met] > 0)
    assert inf <= 2 * finite                # 3 to 19 times with infinite sums formed again
