// Host check of the pooling kernels' tiles (csrc/kern_pool.h): which calls go through LDS, and that what a launch asks for holds
// what its blocks write.  Compiled as HIP for the header's sake; runs no kernel.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include "kern_pool.h"
using namespace mcn;

static PoolGeom geom(int H, int W, int planes, int f, int s, const int (&pad)[4], int method = 0) {
    PoolGeom g = {};
    g.H = H; g.W = W; g.D = planes; g.N = 1; g.Hp = g.Wp = f; g.Sh = g.Sw = s; g.Pt = pad[0]; g.Pl = pad[2]; g.method = method;
    g.Ho = (H + pad[0] + pad[1] - f) / s + 1; g.Wo = (W + pad[2] + pad[3] - f) / s + 1;
    return g;
}

int main() {
    int bad = 0;
    PoolTiles t;
    const int none[4] = {0, 0, 0, 0}, ends[4] = {0, 1, 0, 1};
    // the side of the rule that was measured to be the faster one: H = W, planes, window, stride, through LDS or not
    const int forward[][5] = {{55, 96, 3, 2, 0}, {28, 8192, 3, 2, 0}, {12, 18960, 3, 1, 0}, {55, 12288, 3, 2, 1}, {56, 12288, 3, 1, 1},
                              {112, 4096, 2, 1, 1}, {284, 564, 3, 2, 0}, {13, 256, 3, 2, 0}, {500, 3, 2, 1, 0}};
    for (auto &c : forward)
        if (pool_forward_in_lds(geom(c[0], c[0], c[1], c[2], c[3], none), &t) != (c[4] != 0)) { printf("forward %d, %d planes, %d/%d\n", c[0], c[1], c[2], c[3]); ++bad; }
    const int derivative[][5] = {{55, 96, 3, 2, 0}, {60, 100, 3, 2, 0}, {60, 400, 3, 2, 1}, {55, 12288, 3, 2, 1}, {32, 12, 3, 2, 1}, {89, 1, 3, 2, 0},
                                 {12, 25405, 2, 1, 0}, {224, 512, 2, 1, 0}, {500, 3, 2, 1, 0}, {150, 200, 3, 2, 1}};
    for (auto &c : derivative)
        if (pool_derivative_in_lds(geom(c[0], c[0], c[1], c[2], c[3], ends), &t) != (c[4] != 0)) { printf("derivative %d, %d planes, %d/%d\n", c[0], c[1], c[2], c[3]); ++bad; }
    if (pool_derivative_in_lds(geom(55, 55, 12288, 3, 2, ends, 1), &t)) { printf("the average has no maximum\n"); ++bad; }
    // LDS: within 48 KB (no attribute is asked for), and as much as the blocks use
    for (int H = 1; H <= 700; ++H)
        for (int W = 1; W <= 4200; W = W < 70 ? W + 1 : W * 9 / 8 + 1)
            for (int p = 0; p < 3; ++p) {
                const int pad[4] = {p, p, p, p};
                if (H + 2 * p < 3 || W + 2 * p < 3) continue;
                for (int planes : {1, 3000, 200000}) {
                    if ((double)H * W * planes >= 2147483647.0) continue;
                    const PoolGeom g = geom(H, W, planes, 3, 2, pad);
                    if (!pool_derivative_in_lds(g, &t)) continue;
                    const size_t lds = (size_t)t.xs * 4 + (size_t)t.ws * 5;
                    bool ok = lds <= 48 * 1024 && t.planes >= 1 && (t.strips == 1 ? t.xs >= t.planes * H * W && t.ws >= t.planes * g.Ho * g.Wo : true);
                    for (int i = 0; ok && t.strips > 1 && i < t.strips; ++i) {      // the kernel's ranges of a strip
                        const int s0 = i * t.cols, s1 = s0 + t.cols < W ? s0 + t.cols : W;
                        const int a = s0 + g.Pl - 3 + 2, w0 = a > 0 ? a / 2 : 0;
                        int w1 = (s1 - 1 + g.Pl) / 2 + 1;
                        if (w1 > g.Wo) w1 = g.Wo;
                        if (w1 <= w0) continue;
                        const int c0 = 2 * w0 - g.Pl > 0 ? 2 * w0 - g.Pl : 0, c1 = 2 * (w1 - 1) - g.Pl + 3 < W ? 2 * (w1 - 1) - g.Pl + 3 : W;
                        ok = s0 < s1 && H * (c1 - c0) <= t.xs && g.Ho * (w1 - w0) <= t.ws;
                    }
                    if (!ok && ++bad < 10) printf("LDS: %dx%d, %d planes, pad %d: xs %d ws %d planes %d strips %d cols %d\n", H, W, planes, p, t.xs, t.ws, t.planes, t.strips, t.cols);
                }
            }
    printf(bad ? "BAD %d\n" : "OK\n", bad);
    return bad != 0;
}
