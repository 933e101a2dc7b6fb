// Direct (one result per thread / per wave) kernels: the general fallback that
// accepts every geometry.  They evaluate the sums of Sec. 4.1 of the MatConvNet
// manual (arXiv 1412.4564) and their adjoints (Sec. 2.3.2, Sec. 6.1) term by
// term in fp32.  Lanes run along the first (fastest) array index so that global
// accesses are coalesced.
#pragma once
#include <hip/hip_runtime.h>
#include "geom.h"
#include "fastdiv.h"

namespace mcn {

// y[io,jo,k,n] = b[k] + sum w[fi,fj,fd,k] * x[Sh*io+fi-Pt, Sw*jo+fj-Pl, grp*Df+fd, n]
__global__ __launch_bounds__(256) void direct_forward_kernel(Geom g, const float *__restrict__ x,
                                                             const float *__restrict__ w,
                                                             const float *__restrict__ b,
                                                             float *__restrict__ y, int total, int relu) {
    int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    int io = idx % g.Ho;
    int t = idx / g.Ho;
    int jo = t % g.Wo;
    t /= g.Wo;
    int k = t % g.K;
    int n = t / g.K;
    const int grp = k / g.Kg;
    const float *wk = w + (size_t)k * g.Hf * g.Wf * g.Df;
    const float *xn = x + ((size_t)n * g.D + (size_t)grp * g.Df) * g.H * g.W;
    const int i0 = g.Sh * io - g.Pt, j0 = g.Sw * jo - g.Pl;
    float acc = b ? b[k] : 0.f;
    for (int fd = 0; fd < g.Df; ++fd) {
        for (int fj = 0; fj < g.Wf; ++fj) {
            int j = j0 + fj;
            if (j < 0 || j >= g.W) continue;
            for (int fi = 0; fi < g.Hf; ++fi) {
                int i = i0 + fi;
                if (i < 0 || i >= g.H) continue;
                acc = fmaf(wk[fi + g.Hf * (fj + g.Wf * fd)], xn[i + g.H * (j + (size_t)g.W * fd)], acc);
            }
        }
    }
    y[idx] = relu ? fmaxf(acc, 0.f) : acc;
}

// dzdx[i,j,d,n] = sum over k in group(d), and all (io,fi), (jo,fj) with
// Sh*io+fi-Pt = i, Sw*jo+fj-Pl = j, of w[fi,fj,fd,k] * dzdy[io,jo,k,n].
__global__ __launch_bounds__(256) void direct_backward_data_kernel(Geom g, const float *__restrict__ w,
                                                                   const float *__restrict__ dzdy,
                                                                   float *__restrict__ dzdx, int total) {
    int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    int i = idx % g.H;
    int t = idx / g.H;
    int j = t % g.W;
    t /= g.W;
    int d = t % g.D;
    int n = t / g.D;
    const int grp = d / g.Df, fd = d % g.Df;
    const size_t ysz = (size_t)g.Ho * g.Wo;
    float acc = 0.f;
    for (int kk = 0; kk < g.Kg; ++kk) {
        const int k = grp * g.Kg + kk;
        const float *wk = w + ((size_t)k * g.Df + fd) * g.Hf * g.Wf;
        const float *pk = dzdy + ((size_t)n * g.K + k) * ysz;
        for (int fj = 0; fj < g.Wf; ++fj) {
            int tj = j + g.Pl - fj;
            if (tj < 0) break;            // tj only decreases with fj
            int jo = tj / g.Sw;
            if (tj - jo * g.Sw != 0 || jo >= g.Wo) continue;
            for (int fi = 0; fi < g.Hf; ++fi) {
                int ti = i + g.Pt - fi;
                if (ti < 0) break;
                int io = ti / g.Sh;
                if (ti - io * g.Sh != 0 || io >= g.Ho) continue;
                acc = fmaf(wk[fi + g.Hf * fj], pk[io + (size_t)g.Ho * jo], acc);
            }
        }
    }
    dzdx[idx] = acc;
}

// out[0..total) = 0  (samples of dzdx that no filter tap reaches when a stride exceeds the filter)
__global__ __launch_bounds__(256) void zero_fill_kernel(float *__restrict__ out, int total) {
    const long long lo = (long long)blockIdx.x * 1024, hi = lo + 1024 < total ? lo + 1024 : total;
    for (long long e = lo + threadIdx.x; e < hi; e += 256) out[e] = 0.f;
}

// out[p + plane*(c + C*n)] = bias[c]  (start value of an output whose contributions are written,
// or left out, per stride phase: the convolution transpose with a bias)
__global__ __launch_bounds__(256) void bias_fill_kernel(float *__restrict__ out, const float *__restrict__ bias,
                                                        int plane, int C, int total) {
    const long long lo = (long long)blockIdx.x * 1024, hi = lo + 1024 < total ? lo + 1024 : total;
    for (long long e = lo + threadIdx.x; e < hi; e += 256) out[e] = bias[(e / plane) % C];
}

// out[p + plane*(c + C*n)] += bias[c]
__global__ __launch_bounds__(256) void bias_add_kernel(float *__restrict__ out, const float *__restrict__ bias,
                                                       int plane, int C, int total) {
    const long long lo = (long long)blockIdx.x * 1024, hi = lo + 1024 < total ? lo + 1024 : total;
    for (long long e = lo + threadIdx.x; e < hi; e += 256) out[e] += bias[(e / plane) % C];
}

__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// One wavefront per filter coefficient:
// dzdw[fi,fj,fd,k] = sum_{n,jo,io} x[Sh*io+fi-Pt, Sw*jo+fj-Pl, grp*Df+fd, n] * dzdy[io,jo,k,n]
__global__ __launch_bounds__(256) void direct_backward_filter_kernel(Geom g, const float *__restrict__ x,
                                                                     const float *__restrict__ dzdy,
                                                                     float *__restrict__ dzdw, int total) {
    const int lane = threadIdx.x & 63;
    int e = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (e >= total) return;                 // whole wave leaves together
    int fi = e % g.Hf;
    int t = e / g.Hf;
    int fj = t % g.Wf;
    t /= g.Wf;
    int fd = t % g.Df;
    int k = t / g.Df;
    const int grp = k / g.Kg;
    // valid io range: 0 <= Sh*io + fi - Pt < H
    int lo_i = g.Pt - fi;  lo_i = lo_i > 0 ? (lo_i + g.Sh - 1) / g.Sh : 0;
    int hi_i = g.H - 1 + g.Pt - fi;  hi_i = hi_i < 0 ? -1 : hi_i / g.Sh;  if (hi_i > g.Ho - 1) hi_i = g.Ho - 1;
    int lo_j = g.Pl - fj;  lo_j = lo_j > 0 ? (lo_j + g.Sw - 1) / g.Sw : 0;
    int hi_j = g.W - 1 + g.Pl - fj;  hi_j = hi_j < 0 ? -1 : hi_j / g.Sw;  if (hi_j > g.Wo - 1) hi_j = g.Wo - 1;
    float acc = 0.f;
    for (int n = 0; n < g.N; ++n) {
        const float *xc = x + ((size_t)n * g.D + (size_t)grp * g.Df + fd) * g.H * g.W;
        const float *pc = dzdy + ((size_t)n * g.K + k) * g.Ho * g.Wo;
        for (int jo = lo_j; jo <= hi_j; ++jo) {
            const float *xr = xc + (size_t)g.H * (g.Sw * jo + fj - g.Pl) + (fi - g.Pt);
            const float *pr = pc + (size_t)g.Ho * jo;
            for (int io = lo_i + lane; io <= hi_i; io += 64) acc = fmaf(xr[g.Sh * io], pr[io], acc);
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) dzdw[e] = acc;
}

// ---- bias derivative: dzdb[k] = sum_{n,jo,io} dzdy[io,jo,k,n] ------------------
// Stage 1: the four waves of block (k, s) sum the pieces i = 4s + wave, i + 4S, ... where piece i = (n, c) covers 256 samples of dzdy from
// 256 c on of image n, filter k.  Stage 2 adds the S partials of each k in a fixed order, so the result does not depend on
// scheduling.  S: about 2048 blocks in all, at most one for every BIAS_CHUNK samples of a plane (plan_bias).
//
// RELU, the mask fused with it: Sec. 6.4.1 of the manual, through y = max(0, p) the derivative is dz/dp = [p > 0] dz/dy, and y > 0 exactly
// where p > 0.  One pass reads y and dzdy, writes dzdp = [y > 0] * dzdy (the derivative that the convolution's own backward passes take) and sums
// that.  dzdp may be the array dzdy (each element is read, then written, by one thread).
//
// Bound by HBM.  Four pieces are on their way in a wave, each in 16-byte loads whatever the plane's size and place (the hardware takes
// them at any multiple of 4 bytes).
constexpr int BIAS_CHUNK = 4096, BIAS_PIECE = 256;
// sum of the pieces of wave `wave` (of four) of share s of filter k, in lane 0
template <bool RELU>
__device__ __attribute__((always_inline)) inline float bias_share(const float *__restrict__ y, const float *dzdy, float *dzdp, int HoWo, int K, int N, int pieces,
                                                                  Div32 dPieces, int S, int k, int s, int wave) {
    typedef float Quad __attribute__((ext_vector_type(4), aligned(4)));
    typedef float Quad4 __attribute__((ext_vector_type(4)));
    const int e = 4 * (threadIdx.x & 63);
    const int all = N * pieces, step = 4 * S;
    Quad4 sum[4] = {};
#pragma unroll 1
    for (int i0 = 4 * s + wave; i0 < all; i0 += 4 * step) {
        size_t at[4];
        int left[4];                         // samples from the thread's first one on
        Quad4 v[4], m[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = min(i0 + j * step, all - 1), n = div32(i, dPieces), c = i - n * pieces;
            at[j] = ((size_t)n * K + k) * HoWo + c * BIAS_PIECE + e;
            left[j] = i0 + j * step < all ? HoWo - c * BIAS_PIECE - e : 0;
            v[j] = m[j] = Quad4{0.f, 0.f, 0.f, 0.f};
            if (left[j] >= 4) {
                v[j] = *reinterpret_cast<const Quad *>(dzdy + at[j]);
                if (RELU) m[j] = *reinterpret_cast<const Quad *>(y + at[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (left[j] > 0 && left[j] < 4) {
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    if (u < left[j]) {
                        v[j][u] = dzdy[at[j] + u];
                        if (RELU) m[j][u] = y[at[j] + u];
                    }
            }
            if constexpr (RELU) {
#pragma unroll
                for (int u = 0; u < 4; ++u) v[j][u] = m[j][u] > 0.f ? v[j][u] : 0.f;
                if (left[j] >= 4) *reinterpret_cast<Quad *>(dzdp + at[j]) = v[j];
                else {
#pragma unroll
                    for (int u = 0; u < 3; ++u)
                        if (u < left[j]) dzdp[at[j] + u] = v[j][u];
                }
            }
            sum[j] += v[j];
        }
    }
    const Quad4 q = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    return wave_sum((q[0] + q[1]) + (q[2] + q[3]));
}
template <bool RELU>
__global__ __launch_bounds__(256) void bias_partial_kernel(const float *__restrict__ y, const float *dzdy, float *dzdp, float *__restrict__ part, int HoWo, int K,
                                                           int N, int pieces, Div32 dPieces, int S) {
    const int k = blockIdx.x, s = blockIdx.y, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __shared__ float red[4];
    const float acc = bias_share<RELU>(y, dzdy, dzdp, HoWo, K, N, pieces, dPieces, S, k, s, wave);
    if ((threadIdx.x & 63) == 0) red[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[(size_t)k * S + s] = (red[0] + red[1]) + (red[2] + red[3]);
}
// The same for small output planes, as bias_rows_partial_kernel
__global__ __launch_bounds__(256) void relu_bias_rows_partial_kernel(const float *__restrict__ y, const float *dzdy,
                                                                     float *dzdp, float *__restrict__ part,
                                                                     int KHoWo, int N, int S) {
    const int e = blockIdx.x * 256 + threadIdx.x, s = blockIdx.y;
    if (e >= KHoWo) return;
    float acc = 0.f;
    for (int n = s; n < N; n += S) {
        const size_t a = (size_t)n * KHoWo + e;
        const float m = y[a] > 0.f ? dzdy[a] : 0.f;
        dzdp[a] = m;
        acc += m;
    }
    part[(size_t)s * KHoWo + e] = acc;
}

// Small output planes (down to the 1x1 output of a fully-connected layer): one image of dzdy is
// a contiguous row of K*HoWo values, so threads run along that row and step over the images.
// Stage 1: part[s][e] = sum over images n = s, s+S, ... of dzdy[e + K*HoWo*n], e = p + HoWo*k.
__global__ __launch_bounds__(256) void bias_rows_partial_kernel(const float *__restrict__ dzdy, float *__restrict__ part,
                                                                int KHoWo, int N, int S) {
    const int e = blockIdx.x * 256 + threadIdx.x, s = blockIdx.y;
    if (e >= KHoWo) return;
    float acc = 0.f;
    for (int n = s; n < N; n += S) acc += dzdy[(size_t)n * KHoWo + e];
    part[(size_t)s * KHoWo + e] = acc;
}
// Stage 2: one wavefront per filter adds its S*HoWo partials in a fixed order.
__global__ __launch_bounds__(256) void bias_rows_final_kernel(const float *__restrict__ part, float *__restrict__ dzdb,
                                                              int HoWo, int K, int S) {
    const int lane = threadIdx.x & 63;
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= K) return;                 // whole wave leaves together
    const int KHoWo = K * HoWo, total = S * HoWo;
    float acc = 0.f;
    for (int u = lane; u < total; u += 64) {
        const int s = u / HoWo, p = u - s * HoWo;
        acc += part[(size_t)s * KHoWo + (size_t)k * HoWo + p];
    }
    acc = wave_sum(acc);
    if (lane == 0) dzdb[k] = acc;
}

// One wavefront per filter (one thread that added its S partials one after another took 4.7 us, most of it waiting: 256 filters, S = 8).
__global__ __launch_bounds__(256) void bias_final_kernel(const float *__restrict__ part, float *__restrict__ dzdb,
                                                         int K, int S) {
    const int lane = threadIdx.x & 63, k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= K) return;                 // whole wave leaves together
    float acc = 0.f;
    for (int s = lane; s < S; s += 64) acc += part[(size_t)k * S + s];
    acc = wave_sum(acc);
    if (lane == 0) dzdb[k] = acc;
}

}  // namespace mcn
