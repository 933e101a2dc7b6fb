// Small layers in fp32, one launch a pass: the sums of kern_igemm.h and kern_wgrad.h (MatConvNet manual, arXiv 1412.4564, Sec. 4.1, 6.1) straight
// from the arrays in memory, without packed weights, partial tiles and the passes that make and add them.
//
// What bounds a small layer is launches, and the chain of loads in each: pack, main kernel, fix-up pass, and one or two for the bias, 3 to 12 us one
// behind the other whatever they compute (37x53x16, 3x5x16x24 at stride 2x3, four images, 7.5 million products a pass: eight launches, 44 us).
// Here the chip is filled by cutting the reduction, not the tile: a block owns 64 pixels of 8 filters, its eight waves an eighth of the (channel, tap)
// pairs each, added up in a fixed order through LDS: 26.5 us, three launches, which the host now takes as long to make.  The stride phases of an input derivative are blocks of one launch.  Products are skipped, not
// formed with zeros, where a tap falls into the padding.
#pragma once
#include "kern_igemm_split.h"

namespace mcn {

constexpr int SMALL_K = 8;            // filters of a block
constexpr int SMALL_WAVES = 8;
constexpr int SMALL_VIEWS = 9;        // stride phases at most
constexpr int SMALL_FLIGHT = 8;       // samples on their way to a lane
constexpr int SMALL_PIXELS = 4;      // pixels of a thread in the blocks of 256 (filter derivative)
constexpr int SMALL_HF = 5;           // filter rows at most (filter derivative)
constexpr int SMALL_LDS = 28 * 1024;      // of weights: five blocks to a compute unit

// one stride phase (one in all of a forward pass); weights as in PlainView
struct SmallView {
    int Ho, Wo, pixels;               // pixels: Ho * Wo * N
    int Hf, Wf, Sh, Sw, Pt, Pl;
    int oi0, osi, oj0, osj;
    int wo, wg, wk, wc, wi, wj;
    Div32 dHo, dWo, dT, dHf;
};
struct SmallParams {
    SmallView v[SMALL_VIEWS];
    int H, W, Ctot, Cg, OH, OW, Ktot, Kg, KT, in_bytes, relu;      // KT: blocks of SMALL_K filters per group
    Div32 dKT;
};

__global__ __launch_bounds__(64 * SMALL_WAVES) void small_forward_kernel(SmallParams P, const float *__restrict__ in, const float *__restrict__ w,
                                                                        const float *__restrict__ bias, float *__restrict__ out) {
    extern __shared__ __align__(16) float lds[];       // weights [channel][tap][SMALL_K], then the waves' sums [wave][SMALL_K][64]
    const SmallView &V = P.v[blockIdx.z];
    const int p0 = blockIdx.x * 64;
    if (p0 >= V.pixels) return;
    const int g = div32(blockIdx.y, P.dKT), k0 = (blockIdx.y - g * P.KT) * SMALL_K;
    const int T = V.Hf * V.Wf, M = P.Cg * T, HW = P.H * P.W;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // pixel of the lane
    const int p = p0 + lane;
    const int c1 = div32(p, V.dHo), io = p - c1 * V.Ho, n = div32(c1, V.dWo), jo = c1 - n * V.Wo;
    const int i0 = p < V.pixels ? V.Sh * io - V.Pt : -(1 << 29), j0 = V.Sw * jo - V.Pl;
    for (int e = threadIdx.x; e < M * SMALL_K; e += 64 * SMALL_WAVES) {
        const int m = e >> 3, f = e & 7, c = div32(m, V.dT), t = m - c * T, tj = div32(t, V.dHf), ti = t - tj * V.Hf;
        lds[e] = k0 + f < P.Kg ? w[V.wo + g * V.wg + (k0 + f) * V.wk + c * V.wc + ti * V.wi + tj * V.wj] : 0.f;
    }
    // the wave's pairs of channel and tap, taps fastest
    const int lo = M * wave / SMALL_WAVES, hi = M * (wave + 1) / SMALL_WAVES;
    int c = div32(lo, V.dT), t = lo - c * T, tj = div32(t, V.dHf), ti = t - tj * V.Hf;
    const unsigned base = 4u * (unsigned)(i0 + P.H * j0 + HW * (g * P.Cg + P.Ctot * n));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)in, 0, P.in_bytes, BUFFER_FLAGS);
    float acc[SMALL_K] = {};
    __syncthreads();
    for (int m = lo; m < hi; m += SMALL_FLIGHT) {
        float x[SMALL_FLIGHT];
        bool ok[SMALL_FLIGHT];
#pragma unroll
        for (int u = 0; u < SMALL_FLIGHT; ++u) {
            ok[u] = m + u < hi && (unsigned)(i0 + ti) < (unsigned)P.H && (unsigned)(j0 + tj) < (unsigned)P.W;
            x[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, ok[u] ? base + 4u * (unsigned)(ti + P.H * tj + HW * c) : SLAB_INVALID, 0, 0));
            if (++ti == V.Hf) { ti = 0; if (++tj == V.Wf) { tj = 0; ++c; } }
        }
#pragma unroll
        for (int u = 0; u < SMALL_FLIGHT; ++u) {
            const float4 *q = reinterpret_cast<const float4 *>(lds + SMALL_K * min(m + u, M - 1));
            const float4 a = q[0], b = q[1];
            if (ok[u]) {
                acc[0] = fmaf(a.x, x[u], acc[0]); acc[1] = fmaf(a.y, x[u], acc[1]); acc[2] = fmaf(a.z, x[u], acc[2]); acc[3] = fmaf(a.w, x[u], acc[3]);
                acc[4] = fmaf(b.x, x[u], acc[4]); acc[5] = fmaf(b.y, x[u], acc[5]); acc[6] = fmaf(b.z, x[u], acc[6]); acc[7] = fmaf(b.w, x[u], acc[7]);
            }
        }
    }
    __syncthreads();                                   // the weights have been read
#pragma unroll
    for (int f = 0; f < SMALL_K; ++f) lds[(wave * SMALL_K + f) * 64 + lane] = acc[f];
    __syncthreads();
    // a result a thread: filter `wave` of the block, the lane's pixel
    static_assert(SMALL_WAVES == SMALL_K, "a wave writes a filter's results");
    const int kl = k0 + wave;
    if (kl >= P.Kg || p >= V.pixels) return;
    const int ch = g * P.Kg + kl;
    float s = bias ? bias[ch] : 0.f;
#pragma unroll
    for (int u = 0; u < SMALL_WAVES; ++u) s += lds[(u * SMALL_K + wave) * 64 + lane];
    if (P.relu) s = fmaxf(s, 0.f);
    out[(size_t)(V.oi0 + V.osi * io) + (size_t)P.OH * (V.oj0 + V.osj * jo) + (size_t)P.OH * P.OW * (ch + (size_t)P.Ktot * n)] = s;
}

// dzdw: a block owns one column of taps of one channel for SMALL_K filters, its threads a share of the pixels each; with dzdb (or NULL) further
// blocks for the bias derivative.
struct SmallFilterParams {
    int H, W, D, N, Df, K, Kg, KT, pieces, Hf, Wf, Sh, Sw, Pt, Pl, Ho, Wo, pixels, blocks, x_bytes, y_bytes;      // blocks: of dzdw
    Div32 dHo, dWo, dWf, dDf, dKT, dPieces;
};
// THREADS: 256, or 1024 where each of those has more than SMALL_PIXELS pixels
template <int THREADS>
__global__ __launch_bounds__(THREADS) void small_filter_kernel(SmallFilterParams P, const float *__restrict__ x, const float *__restrict__ dzdy,
                                                           float *__restrict__ dzdw, float *__restrict__ dzdb) {
    __shared__ float red[THREADS / 64][SMALL_HF * SMALL_K];
    const int HoWo = P.Ho * P.Wo, HW = P.H * P.W, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc((void *)dzdy, 0, P.y_bytes, BUFFER_FLAGS);
    auto total = [&](int i) {          // of the waves, in their order
        float s = red[0][i];
#pragma unroll
        for (int u = 1; u < THREADS / 64; ++u) s += red[u][i];
        return s;
    };
    if ((int)blockIdx.x >= P.blocks) {
        // bias_partial_kernel of one share a filter, four waves to a filter
        const int at = (blockIdx.x - P.blocks) * (THREADS / 256) + threadIdx.x / 256, k = min(at, P.K - 1);
        const float s = bias_share<false>(nullptr, dzdy, nullptr, HoWo, P.K, P.N, P.pieces, P.dPieces, 1, k, 0, __builtin_amdgcn_readfirstlane(wave & 3));
        if (lane == 0) red[wave][0] = s;
        __syncthreads();
        if (threadIdx.x % 256 == 0 && at < P.K) dzdb[k] = (red[wave][0] + red[wave + 1][0]) + (red[wave + 2][0] + red[wave + 3][0]);
        return;
    }
    int t = blockIdx.x;
    int q = div32(t, P.dWf);
    const int tj = t - q * P.Wf; t = q;
    q = div32(t, P.dDf);
    const int c = t - q * P.Df; t = q;
    q = div32(t, P.dKT);
    const int k0 = (t - q * P.KT) * SMALL_K, g = q;
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, P.x_bytes, BUFFER_FLAGS);
    float acc[SMALL_HF][SMALL_K] = {};
#pragma unroll 2
    for (int p = threadIdx.x; p < P.pixels; p += THREADS) {
        const int c1 = div32(p, P.dHo), io = p - c1 * P.Ho, n = div32(c1, P.dWo), jo = c1 - n * P.Wo;
        const int i0 = P.Sh * io - P.Pt, j = P.Sw * jo + tj - P.Pl;
        const bool column = (unsigned)j < (unsigned)P.W;
        float y[SMALL_K], xv[SMALL_HF];
        bool ok[SMALL_HF];
#pragma unroll
        for (int f = 0; f < SMALL_K; ++f)
            y[f] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(yrs, k0 + f < P.Kg ? 4u * (unsigned)(io + P.Ho * jo + HoWo * (g * P.Kg + k0 + f + P.K * n)) : SLAB_INVALID, 0, 0));
#pragma unroll
        for (int ti = 0; ti < SMALL_HF; ++ti) {
            ok[ti] = ti < P.Hf && column && (unsigned)(i0 + ti) < (unsigned)P.H;
            xv[ti] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xrs, ok[ti] ? 4u * (unsigned)(i0 + ti + P.H * j + HW * (g * P.Df + c + P.D * n)) : SLAB_INVALID, 0, 0));
        }
#pragma unroll
        for (int ti = 0; ti < SMALL_HF; ++ti)
            if (ok[ti]) {
#pragma unroll
                for (int f = 0; f < SMALL_K; ++f) acc[ti][f] = fmaf(xv[ti], y[f], acc[ti][f]);
            }
    }
#pragma unroll
    for (int ti = 0; ti < SMALL_HF; ++ti)
#pragma unroll
        for (int f = 0; f < SMALL_K; ++f) {
            if (ti >= P.Hf) continue;
            const float s = wave_sum(acc[ti][f]);
            if (lane == 0) red[wave][ti * SMALL_K + f] = s;
        }
    __syncthreads();
    const int f = threadIdx.x % SMALL_K, ti = threadIdx.x / SMALL_K;
    if (ti >= P.Hf || k0 + f >= P.Kg) return;
    dzdw[ti + P.Hf * (tj + P.Wf * (c + (size_t)P.Df * (g * P.Kg + k0 + f)))] = total(threadIdx.x);
}

}  // namespace mcn
