// Spatial pooling (max and average), forward and backward: streaming kernels, one result per
// thread, lanes along the first (fastest) array index.
//
// MatConvNet manual (arXiv 1412.4564) Sec. 4.3: y[io,jo,d,n] is the maximum / the average of x over
// the window rows Sh*io-Pt .. +H'-1, columns Sw*jo-Pl .. +W'-1 of plane (d,n), cropped to the
// array (max: as if padded with -infinity; average: divided by the number of samples inside).
// Sec. 6.3: y = S(x) x, dz/dx = S(x)^T dz/dy; for max pooling S selects one sample per window --
// the first maximum in memory order (rows fastest) -- and the backward pass is written as a
// gather: a sample adds the dzdy of every window that selects it, so no two threads write one
// element and the result does not depend on scheduling.  Which sample a window selects is found
// once per window by pool_argmax_kernel (one byte per window: the position inside the window);
// windows of more than 256 samples take the one-kernel form that rescans the windows.
//
// These kernels move 4-12 bytes per result, so index arithmetic is what they could lose time on:
// the divisions that split a thread's flat index into plane, column and row, and those by the
// strides, are multiplications by reciprocals prepared on the host (exact for every index below 2^31).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fastdiv.h"

namespace mcn {

struct PoolGeom {
    int H, W, D, N;
    int Hp, Wp, Sh, Sw, Pt, Pl;
    int Ho, Wo;
    int method;      // 0 max, 1 average
    Div32 dH, dHo, dSh, dSw;  // exact for every index below 2^31 (fastdiv.h)
    FastDiv64 dIn, dOut;     // by the plane sizes H*W and Ho*Wo
};

// HP, WP > 0: window size known at compile time.  The window's samples are then read with clamped
// addresses and no branches, so that all loads are in flight together (a loop with run-time bounds
// issues them one after the other); samples outside the input are left out by selection, in the same
// order as the loop takes them.
template <int HP, int WP>
__global__ __launch_bounds__(256) void pool_forward_kernel(PoolGeom g, const float *__restrict__ x,
                                                           float *__restrict__ y, unsigned total) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const unsigned plane = div64(idx, g.dOut);
    const int e = (int)(idx - plane * (unsigned)(g.Ho * g.Wo));
    const int jo = div32(e, g.dHo), io = e - jo * g.Ho;
    const float *xp = x + (size_t)plane * g.H * g.W;
    if constexpr (HP > 0) {
        const int oi = g.Sh * io - g.Pt, oj = g.Sw * jo - g.Pl;
        float v[WP][HP];
        bool ok[WP][HP];
#pragma unroll
        for (int fj = 0; fj < WP; ++fj)
#pragma unroll
            for (int fi = 0; fi < HP; ++fi) {
                const int i = oi + fi, j = oj + fj;
                ok[fj][fi] = (unsigned)i < (unsigned)g.H && (unsigned)j < (unsigned)g.W;
                v[fj][fi] = xp[min(max(i, 0), g.H - 1) + g.H * min(max(j, 0), g.W - 1)];
            }
        float r = 0.f;
        int cnt = 0;
#pragma unroll
        for (int fj = 0; fj < WP; ++fj)
#pragma unroll
            for (int fi = 0; fi < HP; ++fi) {
                if (g.method == 0) r = !ok[fj][fi] ? r : cnt == 0 ? v[fj][fi] : fmaxf(r, v[fj][fi]);
                else r += ok[fj][fi] ? v[fj][fi] : 0.f;
                cnt += ok[fj][fi] ? 1 : 0;
            }
        y[idx] = g.method == 0 ? r : r / (float)cnt;
        return;
    }
    const int i0 = max(g.Sh * io - g.Pt, 0), i1 = min(g.Sh * io - g.Pt + g.Hp, g.H);
    const int j0 = max(g.Sw * jo - g.Pl, 0), j1 = min(g.Sw * jo - g.Pl + g.Wp, g.W);
    float r;
    if (g.method == 0) {
        r = xp[i0 + g.H * j0];
        for (int j = j0; j < j1; ++j)
            for (int i = i0; i < i1; ++i) r = fmaxf(r, xp[i + g.H * j]);
    } else {
        float s = 0.f;
        for (int j = j0; j < j1; ++j)
            for (int i = i0; i < i1; ++i) s += xp[i + g.H * j];
        r = s / (float)((i1 - i0) * (j1 - j0));
    }
    y[idx] = r;
}

// The windows that hold sample (i, j): Sh*io - Pt <= i <= Sh*io - Pt + Hp - 1, clipped to the output.
struct WindowRange {
    int io_lo, io_hi, jo_lo, jo_hi;
};
__device__ inline WindowRange windows_of(const PoolGeom &g, int i, int j) {
    WindowRange r;
    const int a = i + g.Pt - g.Hp + g.Sh, b = j + g.Pl - g.Wp + g.Sw;     // ceil((i + Pt - Hp + 1) / Sh) = floor(a / Sh)
    r.io_lo = a > 0 ? div32(a, g.dSh) : 0;
    r.io_hi = min(div32(i + g.Pt, g.dSh), g.Ho - 1);
    r.jo_lo = b > 0 ? div32(b, g.dSw) : 0;
    r.jo_hi = min(div32(j + g.Pl, g.dSw), g.Wo - 1);
    return r;
}

// code[io,jo,plane] = fi + Hp*fj of the first maximum of window (io, jo), (fi, fj) counted from the
// window's uncropped origin.  Needs Hp*Wp <= 256.
template <int HP, int WP>
__global__ __launch_bounds__(256) void pool_argmax_kernel(PoolGeom g, const float *__restrict__ x,
                                                          unsigned char *__restrict__ code, unsigned total) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const unsigned plane = div64(idx, g.dOut);
    const int e = (int)(idx - plane * (unsigned)(g.Ho * g.Wo));
    const int jo = div32(e, g.dHo), io = e - jo * g.Ho;
    const float *xp = x + (size_t)plane * g.H * g.W;
    const int oi = g.Sh * io - g.Pt, oj = g.Sw * jo - g.Pl;
    if constexpr (HP > 0) {
        float v[WP][HP];
#pragma unroll
        for (int fj = 0; fj < WP; ++fj)
#pragma unroll
            for (int fi = 0; fi < HP; ++fi)
                v[fj][fi] = xp[min(max(oi + fi, 0), g.H - 1) + g.H * min(max(oj + fj, 0), g.W - 1)];
        float m = 0.f;
        int best = -1;
#pragma unroll
        for (int fj = 0; fj < WP; ++fj)
#pragma unroll
            for (int fi = 0; fi < HP; ++fi) {
                const bool ok = (unsigned)(oi + fi) < (unsigned)g.H && (unsigned)(oj + fj) < (unsigned)g.W;
                const bool take = ok && (best < 0 || v[fj][fi] > m);
                m = take ? v[fj][fi] : m;
                best = take ? fi + HP * fj : best;
            }
        code[idx] = (unsigned char)best;
        return;
    }
    const int i0 = max(oi, 0), i1 = min(oi + g.Hp, g.H);
    const int j0 = max(oj, 0), j1 = min(oj + g.Wp, g.W);
    float m = xp[i0 + g.H * j0];
    int best = (i0 - oi) + g.Hp * (j0 - oj);
    for (int j = j0; j < j1; ++j)
        for (int i = i0; i < i1; ++i) {
            const float v = xp[i + g.H * j];
            if (v > m) { m = v; best = (i - oi) + g.Hp * (j - oj); }
        }
    code[idx] = (unsigned char)best;
}

// dzdx[i,j] = sum of dzdy over the windows whose code points at (i, j)
// NH, NW > 0: at most NH x NW windows hold one sample (ceil(Hp / Sh) x ceil(Wp / Sw)); their codes and
// derivatives are read with clamped addresses and no branches.
template <int NH, int NW>
__global__ __launch_bounds__(256) void pool_backward_max_coded_kernel(PoolGeom g, const unsigned char *__restrict__ code,
                                                                      const float *__restrict__ dzdy,
                                                                      float *__restrict__ dzdx, unsigned total) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const unsigned plane = div64(idx, g.dIn);
    const int e = (int)(idx - plane * (unsigned)(g.H * g.W));
    const int j = div32(e, g.dH), i = e - j * g.H;
    const size_t pbase = (size_t)plane * g.Ho * g.Wo;
    const WindowRange r = windows_of(g, i, j);
    float acc = 0.f;
    if constexpr (NH > 0) {
        unsigned char c[NW][NH];
        float p[NW][NH];
#pragma unroll
        for (int b = 0; b < NW; ++b)
#pragma unroll
            for (int a = 0; a < NH; ++a) {
                const size_t at = pbase + min(r.io_lo + a, g.Ho - 1) + (size_t)g.Ho * min(r.jo_lo + b, g.Wo - 1);
                c[b][a] = code[at];
                p[b][a] = dzdy[at];
            }
#pragma unroll
        for (int b = 0; b < NW; ++b)
#pragma unroll
            for (int a = 0; a < NH; ++a) {
                const int io = r.io_lo + a, jo = r.jo_lo + b;
                const int fi = i - (g.Sh * io - g.Pt), fj = j - (g.Sw * jo - g.Pl);
                if (io <= r.io_hi && jo <= r.jo_hi && c[b][a] == fi + g.Hp * fj) acc += p[b][a];
            }
        dzdx[idx] = acc;
        return;
    }
    for (int jo = r.jo_lo; jo <= r.jo_hi; ++jo) {
        const int fj = j - (g.Sw * jo - g.Pl);
        for (int io = r.io_lo; io <= r.io_hi; ++io) {
            const int fi = i - (g.Sh * io - g.Pt);
            const size_t a = pbase + io + (size_t)g.Ho * jo;
            if (code[a] == fi + g.Hp * fj) acc += dzdy[a];
        }
    }
    dzdx[idx] = acc;
}

// Max pooling whose windows do not overlap (stride = window size): every sample lies in at most one window,
// so one thread per window reads its samples, finds the first maximum and writes the window's share of dzdx
// (the derivative at the maximum, zero elsewhere) in one pass: x, dzdy and dzdx each move once and no code
// array is needed.  Rows and columns past the last window are cleared by the last windows of each column / row.
template <int HP, int WP>
__global__ __launch_bounds__(256) void pool_backward_max_disjoint_kernel(PoolGeom g, const float *__restrict__ x,
                                                                         const float *__restrict__ dzdy,
                                                                         float *__restrict__ dzdx, unsigned total) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const unsigned plane = div64(idx, g.dOut);
    const int e = (int)(idx - plane * (unsigned)(g.Ho * g.Wo));
    const int jo = div32(e, g.dHo), io = e - jo * g.Ho;
    const size_t base = (size_t)plane * g.H * g.W;
    const float *xp = x + base;
    float *dp = dzdx + base;
    const int oi = HP * io - g.Pt, oj = WP * jo - g.Pl;
    const float p = dzdy[idx];
    float v[WP][HP];
#pragma unroll
    for (int fj = 0; fj < WP; ++fj)
#pragma unroll
        for (int fi = 0; fi < HP; ++fi)
            v[fj][fi] = xp[min(max(oi + fi, 0), g.H - 1) + g.H * min(max(oj + fj, 0), g.W - 1)];
    float m = 0.f;
    int best = -1;
#pragma unroll
    for (int fj = 0; fj < WP; ++fj)
#pragma unroll
        for (int fi = 0; fi < HP; ++fi) {
            const bool ok = (unsigned)(oi + fi) < (unsigned)g.H && (unsigned)(oj + fj) < (unsigned)g.W;
            const bool take = ok && (best < 0 || v[fj][fi] > m);
            m = take ? v[fj][fi] : m;
            best = take ? fi + HP * fj : best;
        }
#pragma unroll
    for (int fj = 0; fj < WP; ++fj)
#pragma unroll
        for (int fi = 0; fi < HP; ++fi)
            if ((unsigned)(oi + fi) < (unsigned)g.H && (unsigned)(oj + fj) < (unsigned)g.W)
                dp[(oi + fi) + g.H * (oj + fj)] = best == fi + HP * fj ? p : 0.f;
    // samples no window reads
    const int i_end = io == g.Ho - 1 ? g.H : oi + HP;          // rows [oi + HP, i_end) below this window
    const int j_end = jo == g.Wo - 1 ? g.W : oj + WP;          // columns [oj + WP, j_end) right of it
    for (int j = max(oj, 0); j < min(oj + WP, g.W); ++j)
        for (int i = oi + HP; i < i_end; ++i) dp[i + g.H * j] = 0.f;
    for (int j = oj + WP; j < j_end; ++j)
        for (int i = max(oi, 0); i < i_end; ++i) dp[i + g.H * j] = 0.f;
}

// ---- overlapping windows through LDS ---------------------------------------------------
// Two kernels that bring the samples of a block into LDS (they are contiguous: whole planes, as many as fit POOL_XS samples, or, of
// larger planes, a strip of columns and the columns that its windows reach beyond it), where the others read every window's
// samples from memory through the caches.
struct PoolTiles {
    int planes, strips, cols;      // planes per block (strips = 1), or strips per plane and columns per strip
    int wcols;                     // forward pass: window columns per strip
    int xs, ws;                    // samples and windows that the LDS arrays hold
    Div32 dna;                     // 3x3 at stride 2: by the pairs of rows of a plane
};
constexpr int POOL_XS = 4096;      // 16 KB of samples; the derivative's five bytes per window come to 5 KB, at most 20 (planes of one column)
inline int64_t pool_blocks(const PoolGeom &g, const PoolTiles &t) { return ((int64_t)g.D * g.N + t.planes - 1) / t.planes * t.strips; }
// false: planes too tall for strips that are wide beside what they share
inline bool pool_tiles(const PoolGeom &g, PoolTiles *t) {
    const int64_t plane = (int64_t)g.H * g.W;
    t->dna = make_div32(((g.H - 1 + g.Pt) >> 1) - (g.Pt >> 1) + 1);
    if (plane <= POOL_XS) {
        const int64_t out = (int64_t)g.Ho * g.Wo;      // may be the larger one (pads)
        t->planes = (int)(POOL_XS / (plane > out ? plane : out));
        const int64_t fill = (int64_t)g.D * g.N / 1024;      // small inputs: rather a thousand blocks than full ones
        if (t->planes > fill) t->planes = (int)fill;
        if (t->planes < 1) t->planes = 1;
        t->strips = 1; t->cols = g.W; t->wcols = g.Wo;
        t->xs = t->planes * (int)plane;
        t->ws = t->planes * g.Ho * g.Wo;
        return true;
    }
    const int halo = 2 * (g.Wp - 1);
    const int most = POOL_XS / g.H - halo;
    if (most < 2 * halo) return false;
    t->planes = 1; t->strips = (g.W + most - 1) / most;
    t->cols = (g.W + t->strips - 1) / t->strips;
    t->strips = (g.W + t->cols - 1) / t->cols;
    t->xs = g.H * (t->cols + halo);
    t->wcols = (g.Wo + t->strips - 1) / t->strips;         // their columns: at most Sw * (wcols - 1) + Wp, checked by the caller
    t->ws = g.Ho * ((t->cols + g.Wp - 2) / g.Sw + 1);      // windows that reach into t->cols columns
    return true;
}

// Where the forward pass goes through LDS: overlapping 2x2 and 3x3 windows over inputs beyond 128 MiB.  Smaller inputs are in the
// caches when the network comes to them, and the nine loads of a window then cost less than the way through LDS (us, loads
// from memory -> through LDS, inputs rotated / the same again; 3x3 at stride 2: 55x55, 96 planes 3.3 -> 5.5 / 3.0 -> 4.8, 28x28, 8192
// planes 13.8 -> 15.8 / 10.6 -> 11.4, 27x27, 32768 planes 39.6 -> 36.4 / 27.8 -> 29.1; 3x3 at stride 1: 12x12, 18960 planes
// 15.3 -> 21.5 / 13.6 -> 18.5); beyond, the memory's accesses count (55x55, 12288 planes 65.6 -> 53.4 / 54.2 -> 41.8; 3x3 at stride 1,
// 56x56, 12288 planes 154 -> 139 / 130 -> 116; 2x2 at stride 1, 112x112, 4096 planes 158 -> 111 / 152 -> 108).  At stride 2 not in strips
// (284x284, 564 planes 75.3 -> 68.7 / 54.1 -> 55.8).
inline bool pool_forward_in_lds(const PoolGeom &g, PoolTiles *t) {
    if (g.Hp != g.Wp || (g.Hp != 2 && g.Hp != 3) || g.Sh >= g.Hp || g.Sw >= g.Wp) return false;
    if ((int64_t)g.H * g.W * g.D * g.N < ((int64_t)1 << 25) || !pool_tiles(g, t)) return false;
    return t->strips == 1 || (g.Sh == 1 && g.Sw == 1 && g.H * (g.Sw * (t->wcols - 1) + g.Wp) <= t->xs);
}

// Where the derivative does: max pooling, 3x3 at stride 2, with enough blocks for the chip, or small ones.  Fewer, large blocks take longer
// than the two passes of the other form (us, two passes -> through LDS, inputs rotated / the same again: 55x55, 96 planes
// 6.4 -> 7.5 / 5.8 -> 6.3, 60x60, 200 planes 8.9 -> 9.7 / 7.3 -> 7.1, but 400 planes 12.9 -> 12.0 / 10.4 -> 8.4, 55x55, 12288 planes
// 191 -> 94 / 166 -> 87; blocks of 32x32 samples, 12 planes 4.2 -> 3.2 / 4.5 -> 3.4).  2x2 at stride 1, with a derivative for every
// sample in four windows, was slower as often as not (12x12, 25405 planes 22.2 -> 27.8, 224x224, 512 planes 156 -> 167).
inline bool pool_derivative_in_lds(const PoolGeom &g, PoolTiles *t) {
    if (g.method != 0 || g.Hp != 3 || g.Wp != 3 || g.Sh != 2 || g.Sw != 2 || !pool_tiles(g, t)) return false;
    return pool_blocks(g, *t) >= 320 || t->xs <= 2048;
}

// n contiguous samples into LDS, eight loads in flight per thread
__device__ inline void pool_stage(float *xs, const float *__restrict__ src, int n) {
    for (int e0 = threadIdx.x; e0 < n; e0 += 8 * 256) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = e0 + u * 256 < n ? src[e0 + u * 256] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (e0 + u * 256 < n) xs[e0 + u * 256] = v[u];
    }
}

// The forward pass (strips of window columns): the samples enter LDS once, coalesced, instead of nine strided loads per window
// (pool_forward_in_lds has the figures).
template <int HP, int WP>
__global__ __launch_bounds__(256) void pool_forward_overlap_kernel(PoolGeom g, PoolTiles t, const float *__restrict__ x, float *__restrict__ y) {
    extern __shared__ float xs[];                                          // [t.xs] samples
    const int HW = g.H * g.W;
    unsigned plane0 = blockIdx.x * (unsigned)t.planes;
    int np = 1, w0 = 0, w1 = g.Wo, c0 = 0, c1 = g.W;                      // window columns, columns loaded
    if (t.strips == 1) {
        np = min((unsigned)t.planes, (unsigned)(g.D * g.N) - plane0);
    } else {
        plane0 = blockIdx.x / (unsigned)t.strips;
        w0 = (int)(blockIdx.x - plane0 * (unsigned)t.strips) * t.wcols;
        w1 = min(w0 + t.wcols, g.Wo);
        if (w0 >= w1) return;
        c0 = max(g.Sw * w0 - g.Pl, 0);
        c1 = min(g.Sw * (w1 - 1) - g.Pl + WP, g.W);
    }
    const int nw1 = g.Ho * (w1 - w0), nw = np * nw1;
    pool_stage(xs, x + (size_t)plane0 * HW + (size_t)g.H * c0, np * g.H * (c1 - c0));
    __syncthreads();
    float *dst = y + (size_t)plane0 * g.Ho * g.Wo + (size_t)g.Ho * w0;
    for (int e = threadIdx.x; e < nw; e += 256) {
        const int pl = np == 1 ? 0 : (int)div64((unsigned)e, g.dOut), rem = e - pl * nw1;
        const int jw = div32(rem, g.dHo), io = rem - jw * g.Ho;
        const int oi = g.Sh * io - g.Pt, oj = g.Sw * (w0 + jw) - g.Pl;
        const float *xp = xs + pl * HW - g.H * c0;
        float r = 0.f;
        int cnt = 0;
#pragma unroll
        for (int fj = 0; fj < WP; ++fj)
#pragma unroll
            for (int fi = 0; fi < HP; ++fi) {
                const float v = xp[min(max(oi + fi, 0), g.H - 1) + g.H * min(max(oj + fj, 0), g.W - 1)];
                const bool ok = (unsigned)(oi + fi) < (unsigned)g.H && (unsigned)(oj + fj) < (unsigned)g.W;
                if (g.method == 0) r = !ok ? r : cnt == 0 ? v : fmaxf(r, v);
                else r += ok ? v : 0.f;
                cnt += ok ? 1 : 0;
            }
        dst[e] = g.method == 0 ? r : r / (float)cnt;
    }
}

// The derivative of max pooling, 3x3 at stride 2, in one pass: every window's maximum is found in LDS, its position and derivative are
// kept there, and the samples gather from them.  Bound by memory: x, dzdy and dzdx move once (and the strips' shared columns
// twice), coalesced, where finding the maxima in one kernel (pool_argmax_kernel, nine strided loads per window) and gathering
// through a byte per window in another move x and dzdy through twice as many instructions (55x55x96, 128 images: 178 -> 82 us,
// 4.1 TB/s).
__global__ __launch_bounds__(256) void pool_backward_max_overlap_kernel(PoolGeom g, PoolTiles t, const float *__restrict__ x,
                                                                        const float *__restrict__ dzdy, float *__restrict__ dzdx) {
    constexpr int HP = 3, WP = 3;
    extern __shared__ float xs[];                                          // [t.xs] samples
    float *ps = xs + t.xs;                                                 // [t.ws] derivatives of the windows
    unsigned char *cs = reinterpret_cast<unsigned char *>(ps + t.ws);      // [t.ws] positions of their maxima
    const int HW = g.H * g.W;
    unsigned plane0 = blockIdx.x * (unsigned)t.planes;
    int np = 1, s0 = 0, s1 = g.W, w0 = 0, w1 = g.Wo, c0 = 0, c1 = g.W;    // columns owned, window columns, columns loaded
    if (t.strips == 1) {
        np = min((unsigned)t.planes, (unsigned)(g.D * g.N) - plane0);
    } else {
        plane0 = blockIdx.x / (unsigned)t.strips;
        s0 = (int)(blockIdx.x - plane0 * (unsigned)t.strips) * t.cols;
        s1 = min(s0 + t.cols, g.W);
        w0 = windows_of(g, 0, s0).jo_lo;
        w1 = max(windows_of(g, 0, s1 - 1).jo_hi + 1, w0);
        c0 = w1 > w0 ? max(g.Sw * w0 - g.Pl, 0) : 0;
        c1 = w1 > w0 ? min(g.Sw * (w1 - 1) - g.Pl + WP, g.W) : 0;
    }
    // all three ranges are contiguous in memory: whole columns of one plane, or whole planes
    const int nx = np * g.H * (c1 - c0), nw1 = g.Ho * (w1 - w0), nw = np * nw1, no1 = g.H * (s1 - s0);
    const float *xsrc = x + (size_t)plane0 * HW + (size_t)g.H * c0;
    const float *psrc = dzdy + (size_t)plane0 * g.Ho * g.Wo + (size_t)g.Ho * w0;
    float *dst = dzdx + (size_t)plane0 * HW + (size_t)g.H * s0;
    const int tid = threadIdx.x;
    pool_stage(xs, xsrc, nx);
    for (int e = tid; e < nw; e += 256) ps[e] = psrc[e];
    __syncthreads();
    for (int e = tid; e < nw; e += 256) {
        const int pl = np == 1 ? 0 : (int)div64((unsigned)e, g.dOut), rem = e - pl * nw1;
        const int jw = div32(rem, g.dHo), io = rem - jw * g.Ho;
        const int oi = g.Sh * io - g.Pt, oj = g.Sw * (w0 + jw) - g.Pl;
        const float *xp = xs + pl * HW - g.H * c0;
        float m = 0.f;
        int best = -1;
#pragma unroll
        for (int fj = 0; fj < WP; ++fj)
#pragma unroll
            for (int fi = 0; fi < HP; ++fi) {
                // clamped columns are loaded ones: a window that reaches past an edge of the plane has the edge's column
                const float v = xp[min(max(oi + fi, 0), g.H - 1) + g.H * min(max(oj + fj, 0), g.W - 1)];
                const bool ok = (unsigned)(oi + fi) < (unsigned)g.H && (unsigned)(oj + fj) < (unsigned)g.W;
                const bool take = ok && (best < 0 || v > m);
                m = take ? v : m;
                best = take ? fi + HP * fj : best;
            }
        cs[e] = (unsigned char)best;
    }
    __syncthreads();
    // 3x3 at stride 2: the samples (2a, 2b) .. (2a+1, 2b+1), counted from the first window's uncropped origin, lie in the
    // windows (a-1, a) x (b-1, b) only, each at a fixed position: a thread gathers four samples from four windows,
    // nine comparisons instead of sixteen with an address each (55x55x96, 128 images: 123 -> 82 us)
    const int a0 = g.Pt >> 1, na = ((g.H - 1 + g.Pt) >> 1) - a0 + 1;                   // pairs of rows
    const int b0 = (s0 + g.Pl) >> 1, nb = ((s1 - 1 + g.Pl) >> 1) - b0 + 1;             // pairs of columns
    const Div32 dna = t.dna;
    for (int e = tid; e < np * na * nb; e += 256) {
        const int q = div32(e, dna), a = a0 + e - q * na;
        const int pl = np == 1 ? 0 : q / nb, b = b0 + q - pl * nb;
        const bool ua = a >= 1 && a - 1 < g.Ho, la = a < g.Ho, ub = b - 1 >= w0 && b - 1 < w1, lb = b >= w0 && b < w1;
        const int at = pl * nw1 + a + g.Ho * (b - w0);
        int c[2][2];
        float p[2][2];                         // [column][row], 0: the window before
        c[0][0] = ua && ub ? cs[at - 1 - g.Ho] : 255; p[0][0] = ua && ub ? ps[at - 1 - g.Ho] : 0.f;
        c[0][1] = la && ub ? cs[at - g.Ho] : 255;     p[0][1] = la && ub ? ps[at - g.Ho] : 0.f;
        c[1][0] = ua && lb ? cs[at - 1] : 255;        p[1][0] = ua && lb ? ps[at - 1] : 0.f;
        c[1][1] = la && lb ? cs[at] : 255;            p[1][1] = la && lb ? ps[at] : 0.f;
        // in the order of the windows: columns, then rows
        const float v00 = (((c[0][0] == 8 ? p[0][0] : 0.f) + (c[0][1] == 6 ? p[0][1] : 0.f)) + (c[1][0] == 2 ? p[1][0] : 0.f)) + (c[1][1] == 0 ? p[1][1] : 0.f);
        const float v10 = (c[0][1] == 7 ? p[0][1] : 0.f) + (c[1][1] == 1 ? p[1][1] : 0.f);
        const float v01 = (c[1][0] == 5 ? p[1][0] : 0.f) + (c[1][1] == 3 ? p[1][1] : 0.f);
        const float v11 = c[1][1] == 4 ? p[1][1] : 0.f;
        const int i = 2 * a - g.Pt, j = 2 * b - g.Pl;
        float *d = dst + pl * no1 + i + g.H * (j - s0);
        const bool r0 = i >= 0, r1 = i + 1 < g.H;
        if (j >= s0) {
            if (r0) d[0] = v00;
            if (r1) d[1] = v10;
        }
        if (j + 1 < s1) {
            if (r0) d[g.H] = v01;
            if (r1) d[g.H + 1] = v11;
        }
    }
}

// One-kernel backward pass: average pooling, and max pooling with windows too large for a byte code.
__global__ __launch_bounds__(256) void pool_backward_kernel(PoolGeom g, const float *__restrict__ x,
                                                            const float *__restrict__ dzdy,
                                                            float *__restrict__ dzdx, unsigned total) {
    const unsigned idx = blockIdx.x * 256u + threadIdx.x;
    if (idx >= total) return;
    const unsigned plane = div64(idx, g.dIn);
    const int e = (int)(idx - plane * (unsigned)(g.H * g.W));
    const int j = div32(e, g.dH), i = e - j * g.H;
    const float *pp = dzdy + (size_t)plane * g.Ho * g.Wo;
    const WindowRange r = windows_of(g, i, j);
    float acc = 0.f;
    if (g.method == 0) {
        const float *xp = x + (size_t)plane * g.H * g.W;
        const float mine = xp[e];
        for (int jo = r.jo_lo; jo <= r.jo_hi; ++jo)
            for (int io = r.io_lo; io <= r.io_hi; ++io) {
                const int i0 = max(g.Sh * io - g.Pt, 0), i1 = min(g.Sh * io - g.Pt + g.Hp, g.H);
                const int j0 = max(g.Sw * jo - g.Pl, 0), j1 = min(g.Sw * jo - g.Pl + g.Wp, g.W);
                // selected iff no sample of the window is larger and none before (i, j) is equal
                bool sel = true;
                for (int jj = j0; jj < j1; ++jj)
                    for (int ii = i0; ii < i1; ++ii) {
                        const float v = xp[ii + g.H * jj];
                        const bool before = jj < j || (jj == j && ii < i);
                        if (v > mine || (before && v == mine)) sel = false;
                    }
                if (sel) acc += pp[io + g.Ho * jo];
            }
    } else {
        for (int jo = r.jo_lo; jo <= r.jo_hi; ++jo) {
            const int j0 = max(g.Sw * jo - g.Pl, 0), j1 = min(g.Sw * jo - g.Pl + g.Wp, g.W);
            for (int io = r.io_lo; io <= r.io_hi; ++io) {
                const int i0 = max(g.Sh * io - g.Pt, 0), i1 = min(g.Sh * io - g.Pt + g.Hp, g.H);
                acc += pp[io + g.Ho * jo] / (float)((i1 - i0) * (j1 - j0));
            }
        }
    }
    dzdx[idx] = acc;
}

}  // namespace mcn
