"""Host time of planning (no GPU): what a call on a new layer waits for before its kernels."""
import ctypes
import os
import subprocess
import time

from paper_1412_4564_amd import binding as B
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def layers(precision, shapes, batch):
    return [B.make_desc((batch, d, w, h), (k, d, f, f), (s, s), (f // 2,) * 4, precision) for h, w, d, f, k, s in shapes]


def query(descs, ops=(B.MCN_OP_FORWARD, B.MCN_OP_BACKWARD_DATA, B.MCN_OP_BACKWARD_FILTER)):
    """Microseconds that size queries of every descriptor take, one after another."""
    refs, size = [ctypes.byref(d) for d in descs], ctypes.c_size_t()
    out, fn = ctypes.byref(size), B.lib().mcn_conv_workspace_size
    start = time.perf_counter()
    for r in refs:
        for op in ops:
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
            best[precision] = min(best[precision], query(layers(precision, SHAPES, batch)))
    print("planning of %d layers: %.0f us, fp32 only %.0f" % (len(SHAPES), best[0], best[2]))
    assert best[0] <= 2.5 * best[2]


def test_a_pass_does_not_wait_for_the_plans_of_another():
    best = {"forward": 1e9, "all": 1e9}
    for batch in range(13, 33, 2):
        best["forward"] = min(best["forward"], query(layers(0, SHAPES, batch), (B.MCN_OP_FORWARD,)))
        best["all"] = min(best["all"], query(layers(0, SHAPES, batch + 1)))
    print("planning of %d layers: forward %.0f us, all passes %.0f" % (len(SHAPES), best["forward"], best["all"]))
    assert best["forward"] <= 0.75 * best["all"]


def test_every_pass_is_planned_once_when_first_asked_for(tmp_path):
    exe = str(tmp_path / "plan_cache_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_1412_4564_amd", "csrc"),
                           "-o", exe, os.path.join(ROOT, "tests", "plan_cache_check.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout[-500:] + r.stderr[-500:]


def test_the_layers_of_a_network_are_remembered():
    best, again = 1e9, 1e9
    for batch in range(40, 60, 5):
        net = [d for b in range(4) for d in layers(0, SHAPES, batch + b)]
        best = min(best, query(net, (B.MCN_OP_FORWARD,)))
        again = min(again, query(net, (B.MCN_OP_FORWARD,)))
    print("forward plans of %d layers: %.0f us, once more %.0f" % (len(net), best, again))
    assert again <= 0.25 * best


def test_stride_phases_of_many_layers():
    """More stride phases (64 a layer) than there is room for: the plans of a layer whose place was taken are made again."""
    descs = [B.make_desc((2, 24 + n, 64, 64), (24 + 16 * n, 24 + n, 9, 8 + n % 3), (8, 8), (0, 0, 0, 0)) for n in range(12)]
    ask = lambda d: (B.mcn_conv_workspace_size(d, B.MCN_OP_BACKWARD_DATA), B.mcn_conv_kernel_name(d, B.MCN_OP_BACKWARD_DATA))
    first = [ask(d) for d in descs]
    assert len(set(first)) > 3
    assert [ask(d) for d in descs] == first and [ask(d) for d in reversed(descs)] == first[::-1]
