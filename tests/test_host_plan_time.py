"""Host time of planning (no GPU): what a call on a new layer waits for before its kernels."""
import ctypes
import time

from paper_1412_4564_amd import binding as B

def layers(precision, shapes, batch):
    return [B.make_desc((batch, d, w, h), (k, d, f, f), (s, s), (f // 2,) * 4, precision) for h, w, d, f, k, s in shapes]


def query(descs, op):
    """Microseconds that one size query of every descriptor takes, one after another."""
    refs, size = [ctypes.byref(d) for d in descs], ctypes.c_size_t()
    out, fn = ctypes.byref(size), B.lib().mcn_conv_workspace_size
    start = time.perf_counter()
    for r in refs:
        fn(r, op, out)
    return 1e6 * (time.perf_counter() - start)


# 1x1 to 11x11 filters, strides 1 to 4, deep and shallow: layers whose filter derivative has a plan in three planes
SHAPES = [(28, 28, 512, 1, 128, 1), (14, 14, 256, 1, 512, 1), (16, 16, 32, 5, 32, 1), (27, 27, 48, 5, 128, 1), (56, 56, 128, 4, 256, 2),
          (30, 30, 64, 7, 96, 1), (55, 55, 3, 11, 96, 4), (20, 24, 112, 2, 200, 1), (7, 7, 512, 1, 512, 1), (13, 13, 96, 6, 72, 3)]


def test_planning_in_three_planes_is_not_much_longer_than_in_fp32():
    """A new layer's plans with the three-plane kernels against those without (MCN_PREC_FP32_PLAIN): a search of the slab's pitches for
    every tile tried made it four to five times as long."""
    best = {0: 1e9, 2: 1e9}
    for batch in range(1, 13):                 # other descriptors every time: none is remembered
        for precision in best:
            best[precision] = min(best[precision], query(layers(precision, SHAPES, batch), 2))
    print("planning of %d layers: %.0f us, fp32 only %.0f" % (len(SHAPES), best[0], best[2]))
    assert best[0] <= 2.5 * best[2]
