// Filter derivative of fp32 operands on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16).
//
// The sum is that of kern_wgrad.h (MatConvNet manual, arXiv 1412.4564, Sec. 6.1, dz/dF = phi(x)^T dz/dY summed over the
// batch), in fp32 precision as in kern_igemm_split.h: every operand is held on chip as three bf16 planes whose (scaled) sum it
// is exactly, a product is six MFMAs, and the three scales have accumulators of their own.
//
// GEMM view OUT[k][r] = sum_p DY[k][p] * PATCH[r][p], r = fi + Hf*(fj + Wf*c).  One MFMA takes 16 terms of the reduction, a lane
// eight of them (an octet): 4 consecutive rows of one column in 2 images, images fastest.  A pair of images is then one
// 32-bit word of a plane, and an octet of x may start at any row (filter row fi shifts it by fi words): the LDS reads words at
// any 4-byte boundary at 128 bytes a cycle (ds_read2_b32; 16-byte reads that are not aligned take eleven times as long), and
// the slab is stored once.  With 8 rows of one image an octet would start at odd halves of a word and the slab have to be stored
// Hf times; with 8 images the memory would be read in runs of a quarter of a line.
//   dzdy tile  [filter][octet][plane] in 16-byte words
//   x slab     [plane][channel][image pair][column][row phase][row] in 32-bit words (pair of images); row phase: vertical stride
// A unit is a patch of TI rows x MC columns x 2*NP images, and shares its halo columns with the unit before it (ring of columns).
// Four staging waves fetch and split the next unit while eight computing waves of 32*MK filters x 32 coefficients multiply; the
// split's vector instructions run beside the bf16 MFMAs (6 a product slow a loop of products by 10 %, 64 per 12 products in other
// waves by 5 %), which they do not on the fp32 matrix core.
//
// What bounds it: the matrix core at the clock that its power leaves (27x27x96, 5x5x48x256 in two groups, 128 images: 285 us at 1.9 GHz, 220
// without operand reads and staging, 250 without staging; the fp32 kernel 556), then the staging waves' vector instructions where
// few coefficients share a sample (28x28x512, 1x1x512x128, 64 images: 66 us, fp32 103; 4x4 at stride 2, 56x56x128, 256 filters, 32
// images: 205, fp32 276).  Hence
//  * every octet is requested as soon as the same octet of the unit before has been split, without branches between the requests
//    (with all requests behind the last write, or branches that make the compiler wait for all of them: 374 to 490 us);
//  * the waves wait for one another through counters in LDS, a unit ahead, and not at barriers;
//  * where an octet lies in the slab is read across lanes from registers: from a table in LDS, every step began with a wait for all of
//    its operands (330 us).
// Tried and dropped: rows of x by 16-byte loads (strides 1, 2, 4; 262 -> 329 us on 11x11 filters at stride 4: fewer waves then split
// more each); a branch around the zeroing of rows past the plane (+3 %); wave priorities (+6 %); two units of registers on their
// way (37 of them spilled).
//
// Schedules, tiles and the fix-up pass: kern_wgrad.h.
#pragma once
#include "kern_wgrad.h"

namespace mcn {

constexpr int WGS_STAGE_WAVES = 4;

struct WgradSplitParams : WgradParams {
    // strides in elements (rows are adjacent): image, channel, column
    long long xtot, ytot;            // elements of x and dzdy
    int xsn, xsc, xsj, ysn, ysc, ysj;
    int NP, IB;                      // image pairs per unit, blocks of 2*NP images
    int TIQ, NO;                     // row quads per patch column, octets per unit = TIQ*MC*NP (even, at most 32)
    int PYW;                         // words of 3 planes per filter in LDS (odd)
    int NPH, XQ;                     // row phases of the slab, row quads per phase
    int PHP, COLP, MPP, CHP, XPL;    // slab pitches in 32-bit words: row phase, column, image pair, channel, plane
    int RC;                          // columns of the slab ring: two units' worth
    int step;                        // columns that a unit adds to the one before it in the same sweep (SC: all of them)
    int YW, XW1;                     // staged words: dzdy per unit, slab per column (NCH channels)
    int counts;                      // byte offset of four counters in LDS
    int XL;                          // rows of the slab before the row of x that meets filter row Pt (kern_wgrad_bf16.h: the next multiple of 4, else Pt)
    Div32 dRB, dCC, dXW1, dXQ, dNPH, dNP;
};

// ---- results that are not finite (see kern_igemm_split.h) --------------------------------
// Part `part` of `parts` of a lane's coefficient (g, k, r), summed as Sec. 6.1 writes it, in fp32: the terms of a coefficient go by runs of
// at most 64 rows of a column, dealt among its parts.  All lanes of a wave call it together; stop(nan), after every run: whether a part of the
// coefficient is NaN by now, and with it the sum.  Bound by the latency of its loads: 8 rows are on their way at a time.
template <class Stop>
__device__ inline float wgrad_plain_part(const WgradSplitParams &P, const float *x, const float *dzdy, int g, int k, int r, int part, int parts, bool on, Stop stop) {
    typedef float Quad __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int RUN = 64;
    const int T = P.Hf * P.Wf, c = r / T, tap = r - c * T, fj = tap / P.Hf, fi = tap - fj * P.Hf;
    // rows and columns of dzdy that meet a sample inside the array
    const int i0 = max(0, (P.Pt - fi + P.Sh - 1) / P.Sh), i1 = P.H - 1 + P.Pt < fi ? 0 : min(P.Ho, (P.H - 1 + P.Pt - fi) / P.Sh + 1);
    const int j0 = max(0, (P.Pl - fj + P.Sw - 1) / P.Sw), j1 = P.W - 1 + P.Pl < fj ? 0 : min(P.Wo, (P.W - 1 + P.Pl - fj) / P.Sw + 1);
    const int runs = max(0, i1 - i0 + RUN - 1) / RUN, cols = max(0, j1 - j0);
    const unsigned all = on ? P.N * cols * runs : 0;
    const float *const x0 = x + (size_t)(g * P.Cg + c) * P.xsc + ((ptrdiff_t)(fj - P.Pl) * P.xsj + (fi - P.Pt)), *const y0 = dzdy + (size_t)(g * P.Kg + k) * P.ysc;
    float s = 0.f;
    bool done = false;
#pragma unroll 1
    for (unsigned q = part;; q += parts) {
        const bool more = q < all && !done;
        if (!__any(more)) break;
        if (more) {
            const int line = (int)q / runs, n = line / cols, jo = j0 + line - n * cols, io0 = i0 + RUN * ((int)q - line * runs), last = min(io0 + RUN, i1) - 1;
            const float *const xc = x0 + (size_t)n * P.xsn + (ptrdiff_t)jo * P.Sw * P.xsj, *const yc = y0 + (size_t)n * P.ysn + (size_t)jo * P.ysj;
            int io = io0;
            if (P.Sh == 1 && i1 - i0 >= 4) {
                // two fours of rows that end with the run at the latest: rows that they share count once
#pragma unroll 1
                for (; io <= last; io += 8) {
                    const int a[2] = {min(io, last - 3), min(io + 4, last - 3)};
                    Quad xq[2], yq[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) { xq[e] = *(const Quad *)(xc + a[e]); yq[e] = *(const Quad *)(yc + a[e]); }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float next = fmaf(xq[e / 4][e % 4], yq[e / 4][e % 4], s);
                        s = a[e / 4] + e % 4 >= io + e / 4 * 4 ? next : s;
                    }
                }
            }
#pragma unroll 1
            for (; io <= last; io += 4) {
                float xv[4], yv[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = min(io + e, last);
                    xv[e] = xc[i * P.Sh]; yv[e] = yc[i];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float next = fmaf(xv[e], yv[e], s);
                    s = io + e <= last ? next : s;
                }
            }
        }
        done |= stop(s != s);
    }
    return s;
}

// How many of `threads` (a power of two) sum one of m results together, a power of two.
__device__ inline int repair_parts(int threads, int m) { return 1 << (31 - __clz(threads / m)); }

// By a wave: the coefficients (g, k, r) of the lanes that ask for it.  The lanes are shared out among them.
__device__ __attribute__((always_inline)) inline float wave_sum_again(const WgradSplitParams &P, const float *x, const float *dzdy, int g, int k, int r, bool again) {
    const int lane = threadIdx.x & 63;
    const unsigned long long which = __ballot(again);
    // lane's coefficient is that of the j-th lane that has one
    const int m = __popcll(which), parts = repair_parts(64, m), j = lane / parts, p = lane - j * parts;
    unsigned long long left = which;
    for (int i = 0; i < j; ++i) left &= left - 1;
    const int from = left ? __ffsll((long long)left) - 1 : 0;
    const unsigned long long together = (parts == 64 ? ~0ull : (1ull << parts) - 1) << (j * parts);
    float val = wgrad_plain_part(P, x, dzdy, g, __shfl(k, from), __shfl(r, from), p, parts, j < m,
                                 [&](bool nan) __attribute__((always_inline)) { return (__ballot(nan) & together) != 0; });
    for (int h = parts >> 1; h > 0; h >>= 1) val += __shfl_xor(val, h);
    const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(which >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)which, 0u));
    return __shfl(val, rank * parts);
}

// In the fix-up pass: of n stored results, where(i, &k, &r) says which and whether there is one, those that are not finite are summed
// again by the block's 512 threads, shared out evenly.  Times at most and in the mean over channels and places in the plane: 27x27x96,
// 5x5x48x256 in two groups, 128 images (0.31 ms): one NaN in x 1.0, 0.5 ms, in dzdy 1.0, 0.8, one inf 1.7, 0.9 and 1.0, 1.0, all NaN 0.3, +inf
// everywhere 13; 28x28x512, 1x1x512x128, 64 images (0.07 ms): one NaN 0.2 at most, one inf 0.2 and 0.6; 227x227x3, 11x11x3x96 at stride 4, 128
// images (0.25 ms), where the results of few blocks meet it: one NaN 0.9 and 0.6, one inf 2.2 and 6.4; 14x14x512, 5x5x512x512, 32 images (0.46 ms):
// one NaN 5.7 and 0.8, one inf 9.8 and 0.8.  At most 32 or 64 results at a time, each by more threads: the same but for all NaN, 0.6 -> 1.1 and 1.7.
// NAN_ONLY: infinite ones stay (kern_wgrad_bf16.h).
template <bool NAN_ONLY>
struct RepairSums {
    static constexpr bool on = true;
    static __device__ bool again(float v) { return NAN_ONLY ? v != v : not_finite(v); }
    WgradSplitParams S;
    const float *x, *dzdy;
    template <class Where>
    __device__ void operator()(int g, int n, Where where, const float *rbias, int relu, float *out) const {
        __shared__ float part[512];
        __shared__ int list[512], dead[512], found;
        const int tid = threadIdx.x;
#pragma unroll 1
        for (int c0 = 0; c0 < n; c0 += 512) {
            int k = 0, r = 0;
            if (tid == 0) found = 0;
            dead[tid] = 0;
            __syncthreads();
            if (c0 + tid < n && where(c0 + tid, &k, &r) && again(*(volatile float *)(out + (size_t)(g * S.Kg + k) * S.R + r))) list[atomicAdd(&found, 1)] = c0 + tid;
            __syncthreads();
            const int m = found;
            if (m > 0) {
                // neighbours take neighbouring coefficients, whose samples share lines of memory
                const int parts = repair_parts(512, m), M = 512 / parts, j = tid & (M - 1), p = tid / M;
                const bool mine = j < m;
                where(list[mine ? j : 0], &k, &r);
                part[tid] = wgrad_plain_part(S, x, dzdy, g, k, r, p, parts, mine, [&](bool nan) __attribute__((always_inline)) {
                    if (nan) dead[j] = 1;
                    return *(volatile int *)&dead[j] != 0;
                });
#pragma unroll 1
                for (int h = parts >> 1; h > 0; h >>= 1) {
                    __syncthreads();
                    if (p < h) part[tid] += part[tid + h * M];
                }
                if (mine && p == 0) {
                    float v = dead[j] ? __uint_as_float(0x7fc00000u) : part[tid];
                    if (rbias) v += rbias[r];
                    out[(size_t)(g * S.Kg + k) * S.R + r] = relu ? fmaxf(v, 0.f) : v;
                }
            }
            __syncthreads();
        }
    }
};

// YT, XT: 16-byte words (octets) of dzdy and of new slab columns that a staging thread brings per unit, at most.
// LINEAR: 1x1 filters at stride 1 whose output has the rows of x: octets of x lie in memory like those of dzdy
template <int WK, int WR, int MK, int YT, int XT, bool LINEAR>
__global__ __launch_bounds__(64 * (WK * WR + WGS_STAGE_WAVES), 3) void wgrad_split_kernel(WgradSplitParams P, const float *__restrict__ x,
                                                                                       const float *__restrict__ dzdy,
                                                                                       const float *__restrict__ rbias, float *out,
                                                                                       float *__restrict__ part) {
    constexpr int NT = 64 * WK * WR;               // computing threads
    constexpr int NL = 64 * WGS_STAGE_WAVES;       // staging threads
    constexpr int TK = WK * MK * 32, TR = WR * 32;
    const int NU = P.NU;
    const int T = P.Hf * P.Wf;
    const int YB = TK * P.PYW * 48;                // bytes per buffer of dzdy

    extern __shared__ __align__(16) float lds[];
    char *const ybuf = reinterpret_cast<char *>(lds), *const xbuf = ybuf + 2 * YB;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int vb;
    long long ub, ue;
    if (P.nchunks > 0) {
        vb = wg_chunk_virtual_block(blockIdx.x, gridDim.x);
        if (vb >= P.nblocks) return;
        const int tile = vb % P.tiles, chunk = vb / P.tiles;
        ub = (long long)tile * NU + sk_begin(P.walk, chunk);
        ue = (long long)tile * NU + sk_begin(P.walk, chunk + 1);
    } else {
        vb = sk_virtual_block(blockIdx.x, P.nblocks);
        ub = sk_begin(P.walk, vb);
        ue = sk_begin(P.walk, vb + 1);
    }
    if (ub >= ue) return;
    const int nunits = (int)(ue - ub);
    int t = sk_tile(P.walk, ub, NU), uu = (int)(ub - (long long)t * NU);

    // Units done, in waves: written by the staging waves, read by the computing ones.  The waves wait for one another through these two
    // and not at barriers: the two computing waves of a SIMD then drift apart, and one multiplies while the other waits for the
    // first operands of a unit.  The LDS executes a wave's accesses in order, so a count follows what it counts.
    typedef __attribute__((address_space(3))) int LdsInt;
    LdsInt *const written = (LdsInt *)(ybuf + P.counts), *const read = written + 2;      // of even units, of odd ones
    if (tid < 4) written[tid] = 0;
    __syncthreads();
    auto count = [&](LdsInt *c) __attribute__((always_inline)) {
        if (lane == 0) asm volatile("ds_add_u32 %0, %1" ::"v"((unsigned)(size_t)c), "v"(1) : "memory");
    };
    auto await = [&](LdsInt *c, int n) __attribute__((always_inline)) {
        while (__builtin_amdgcn_readfirstlane(*(volatile LdsInt *)c) < n) __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
    };
    // Units follow one another along the columns of a block of rows ("sweep"), so that a unit shares all but `step` of its slab
    // columns with the one before it; they stay where they are, in a ring of RC columns.
    const int RCB = 4 * P.RC * P.COLP;             // ring in bytes

    if (wave >= WK * WR) {
        // ---- the waves that fetch and split ---------------------------------------------------
        const int ltid = tid - NT;
        // What the thread brings: dzdy words (filter, line, quad), quads fastest; slab words (column, channel, image pair, row phase,
        // quad) of a unit's last `step` columns.  y_at: filter, first row, column and first image, a byte each, to be compared with
        // their limits at once.  What a unit does not have is requested out of range and reads as zero: no branches, so that the
        // waits for a word leave the younger ones on their way.
        constexpr unsigned GUARD = 0x80808080u;
        unsigned y_at[YT];
        int y_off[YT];
#pragma unroll
        for (int s = 0; s < YT; ++s) {
            const int q = ltid + NL * s, k = q / P.NO, o = q - k * P.NO, line = o / P.TIQ, m = line / P.MC, row = 4 * (o - line * P.TIQ), col = line - m * P.MC;
            y_at[s] = q < P.YW ? (unsigned)(k | row << 8 | col << 16 | m << 25) : 0x7fu << 24;        // 127th image: never there
            y_off[s] = 4 * (k * P.ysc + col * P.ysj + row + 2 * m * P.ysn);
        }
        const int XW = P.step * P.XW1;
        struct Word { int col, c, row, img, lds; };
        auto slab_word = [&](int q) __attribute__((always_inline)) {
            Word w;
            w.col = div32(q, P.dXW1); q -= w.col * P.XW1;
            const int a = div32(q, P.dXQ), quad = q - a * P.XQ, b = div32(a, P.dNPH), ph = a - b * P.NPH;
            w.c = div32(b, P.dNP);
            const int m = b - w.c * P.NP;
            w.img = 2 * m;
            w.row = 4 * quad * P.Sh + ph;
            w.lds = 4 * (w.c * P.CHP + m * P.MPP + ph * P.PHP + 4 * quad);
            return w;
        };
        Word xw[XT];
#pragma unroll
        for (int s = 0; s < XT; ++s) {
            const int q = ltid + NL * s;
            xw[s] = slab_word(q);
            if (q >= XW) xw[s].c = 0x40000000;
        }
        int klim = 0, nch = 0, xch = 0, ych = 0;
        auto set_tile = [&](int tt) __attribute__((always_inline)) {
            const int rt = tt % P.RT; tt /= P.RT;
            const int kt = tt % P.KT, g = tt / P.KT;
            const int r_lo = rt * TR, r_hi = min(r_lo + TR, P.R), c_lo = r_lo / T;
            nch = (r_hi - 1) / T - c_lo + 1;
            klim = min(P.Kg - kt * TK, TK);
            xch = g * P.Cg + c_lo;
            ych = g * P.Kg + kt * TK;
        };
        struct Place { int io0, jo0, n0, rows; bool start; };          // of a unit; start: it shares no column with the one before
        bool fresh = true;                 // the next unit to request is the block's first one of its tile
        auto place = [&]() __attribute__((always_inline)) {
            const int jr = div32(uu, P.dCC), jc = uu - jr * P.CC, ib = div32(jr, P.dRB), rb = jr - ib * P.RB;
            return Place{rb * P.TI, jc * P.MC, ib * 2 * P.NP, min(P.TI, P.Ho - rb * P.TI), fresh || jc == 0};
        };
        auto x_rsrc = [&](int n0, int ch, bool on) __attribute__((always_inline)) {
            const long long xb = (long long)n0 * P.xsn + (long long)ch * P.xsc, xl = 4 * (P.xtot - xb);
            return __builtin_amdgcn_make_buffer_rsrc((void *)(x + xb), 0, !on ? 0 : xl > 0x7fffffff ? 0x7fffffff : (int)xl, BUFFER_FLAGS);
        };
        // first: the unit's column that the words' column 0 is
        auto load_x = [&](float (&v)[2][4], const Word &w, const Place &u, int first, int nch, __amdgpu_buffer_rsrc_t xrs) __attribute__((always_inline)) {
            const int i0 = w.row + u.io0 * P.Sh - P.Pt, j = w.col + first + u.jo0 * P.Sw - P.Pl;
            // of a word that is not there (channel 0x40000000, columns far outside) some number that is not used: unsigned, so that it may wrap
            const unsigned off = 4u * ((unsigned)i0 + (unsigned)j * (unsigned)P.xsj + (unsigned)w.c * (unsigned)P.xsc + (unsigned)(w.img * P.xsn));
            const bool ok = (w.c < nch) & ((unsigned)j < (unsigned)P.W);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const bool oki = ok & (w.img + i < P.N - u.n0);
                if constexpr (LINEAR) {
                    const uintx4 q = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(xrs, (oki & (w.row < u.rows)) ? off + 4u * (unsigned)(i * P.xsn) : SLAB_INVALID, 0, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[i][e] = __uint_as_float(q[e]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[i][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                            xrs, (oki & ((unsigned)(i0 + e * P.Sh) < (unsigned)P.H)) ? off + 4u * (unsigned)(e * P.Sh + i * P.xsn) : SLAB_INVALID, 0, 0));
                }
            }
        };
        // col: where the words' column 0 goes in the ring, in bytes
        auto put_x = [&](const float (&v)[2][4], const Word &w, int col) __attribute__((always_inline)) {
            unsigned h[4], m[4], l[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) split_bf16x3(v[0][e], v[1][e], &h[e], &m[e], &l[e]);
            if (w.c < 0x40000000) {
                const unsigned at = (unsigned)(col + 4 * w.col * P.COLP), at1 = at - (unsigned)RCB;
                unsigned *dst = reinterpret_cast<unsigned *>(xbuf + (w.lds + (int)min(at, at1)));
#pragma unroll
                for (int e = 0; e < 4; ++e) { dst[e] = h[e]; dst[P.XPL + e] = m[e]; dst[2 * P.XPL + e] = l[e]; }
            }
        };
        // What is on its way: one unit, every word of it requested as soon as the same word of the unit before has been written, so
        // that it has a unit's time to come.
        uintx4 yv[YT][2];
        float xv[XT][2][4];
        float xe[2][2][4];                 // a sweep's first unit: the columns that a unit otherwise finds in place
        Place cur = {};                    // where that unit is
        int ring = 0;                      // where its first new column goes, in bytes
        auto stage = [&](int b, bool put, bool get) __attribute__((always_inline)) {
            const Place in = place();      // the unit to request
            const int first = P.SC - P.step;
            const int extra = first * P.XW1;
            int next_ring = ring;
            if (put && cur.start) { next_ring += 4 * first * P.COLP; if (next_ring >= RCB) next_ring -= RCB; }
            auto extra_word = [&](int s) __attribute__((always_inline)) {
                Word w = slab_word(ltid + NL * s);
                if (ltid + NL * s >= extra) w.c = 0x40000000;
                return w;
            };
            const long long yb = (long long)in.n0 * P.ysn + (long long)ych * P.ysc, yl = 4 * (P.ytot - yb);
            const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc((void *)(dzdy + yb), 0, !get ? 0 : yl > 0x7fffffff ? 0x7fffffff : (int)yl, BUFFER_FLAGS);
            const int y0 = 4 * (in.io0 + in.jo0 * P.ysj);
            const unsigned lim = GUARD | (unsigned)(klim - 1) | (unsigned)(in.rows - 1) << 8 | (unsigned)(min(P.Wo - in.jo0, 127) - 1) << 16 | (unsigned)(min(P.N - in.n0, 127) - 1) << 24;
            char *const ybl = ybuf + b * YB;
#pragma unroll
            for (int s = 0; s < YT; ++s) {
                if (put) {
                    unsigned h[4], m[4], l[4];
                    const int nv = cur.rows - (int)(y_at[s] >> 8 & 255);     // rows past the patch's last one are those of the next column: they must not count
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        split_bf16x3(e < nv ? __uint_as_float(yv[s][0][e]) : 0.f, e < nv ? __uint_as_float(yv[s][1][e]) : 0.f, &h[e], &m[e], &l[e]);
                    const int q = ltid + NL * s;
                    if (q < P.YW) {
                        uintx4 *dst = reinterpret_cast<uintx4 *>(ybl + (q + (int)(y_at[s] & 255) * (P.PYW - P.NO)) * 48);
                        dst[0] = uintx4{h[0], h[1], h[2], h[3]}; dst[1] = uintx4{m[0], m[1], m[2], m[3]}; dst[2] = uintx4{l[0], l[1], l[2], l[3]};
                    }
                }
                const unsigned left = lim - y_at[s], off = (unsigned)(y_off[s] + y0);
                yv[s][0] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(yrs, (left & GUARD) == GUARD ? off : SLAB_INVALID, 0, 0));
                yv[s][1] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(yrs, (left & (left - (1u << 24)) & GUARD) == GUARD ? off + 4u * (unsigned)P.ysn : SLAB_INVALID, 0, 0));
            }
            const __amdgpu_buffer_rsrc_t xrs = x_rsrc(in.n0, xch, get);
#pragma unroll
            for (int s = 0; s < XT; ++s) {
                if (put) put_x(xv[s], xw[s], next_ring);
                load_x(xv[s], xw[s], in, first, nch, xrs);
            }
            if (extra > 0) {
                if (put && cur.start) {
#pragma unroll
                    for (int s = 0; s < 2; ++s) put_x(xe[s], extra_word(s), ring);
                }
                // the youngest requests: no wait for other words has to allow for them
                if (get && in.start) {
#pragma unroll
                    for (int s = 0; s < 2; ++s) load_x(xe[s], extra_word(s), in, 0, nch, xrs);
                }
            }
            if (put) {
                ring = next_ring + 4 * P.step * P.COLP;
                if (ring >= RCB) ring -= RCB;
            }
            cur = in;
            fresh = false;
            if (++uu == NU && ++t < P.tiles) { uu = 0; fresh = true; set_tile(t); }
        };
        set_tile(t);
        stage(0, false, true);
        for (int it = 0; it < nunits; ++it) {        // unit it is written while unit it - 1 is computed
            await(read + (it & 1), (it >> 1) * (WK * WR));
            stage(it & 1, true, it + 1 < nunits);
            count(written + (it & 1));
        }
        return;
    }

    // ---- the computing waves -------------------------------------------------------------------
    const int wk = wave % WK, wr = wave / WK;
    floatx16 acc[MK], sum8[MK], sum16[MK];
    int c_rt = 0, c_kt = 0, c_g = 0, roff = 0, rcol = 0;      // roff, rcol: where the lane's coefficient is in the slab, in bytes, but for the column; its column
    auto set_tile = [&](int tt) __attribute__((always_inline)) {
        c_rt = tt % P.RT; tt /= P.RT;
        c_kt = tt % P.KT; c_g = tt / P.KT;
        const int r = c_rt * TR + wr * 32 + l32, c_lo = c_rt * TR / T;
        roff = rcol = 0;
        if (r < P.R) {
            const int c = r / T, tap = r - c * T, fj = tap / P.Hf, fi = tap - fj * P.Hf, a = fi / P.Sh;
            roff = 4 * ((c - c_lo) * P.CHP + (fi - a * P.Sh) * P.PHP + a);
            rcol = 4 * fj * P.COLP;
        }
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mk][v] = sum8[mk][v] = sum16[mk][v] = 0.f;
    };
    // Lane o: where octet o of a unit starts in the slab, in bytes: its column and the rest apart.  An octet is (line, rows 4*q on),
    // line = (image pair, column).  Read across lanes: a table in LDS would make every step wait for all of its operands.
    int oct_col, oct_at;
    {
        const int line = lane / P.TIQ, q = lane - line * P.TIQ, m = line / P.MC, dc = line - m * P.MC;
        oct_col = 4 * dc * P.Sw * P.COLP;
        oct_at = 4 * (m * P.MPP + 4 * q);
    }
    typedef bf16x8 OpA[MK];
    OpA ah, am, al;
    bf16x8 bh, bm, bl;
    const int aoff = ((wk * MK * 32 + l32) * P.PYW + half) * 48, amk = 32 * P.PYW * 48;
    const int xpl = P.XPL * 4;
    const char *ya = ybuf;            // the lane's octet of the next operands
    const char *xa = xbuf;
    int ring = 0;                     // the unit's first column, in bytes
    auto load_a = [&](OpA &a, int pl) __attribute__((always_inline)) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) a[mk] = *reinterpret_cast<const bf16x8 *>(ya + mk * amk + pl * 16);
    };
    auto load_b = [&](bf16x8 &b, int pl) __attribute__((always_inline)) {
        const unsigned *p = reinterpret_cast<const unsigned *>(xa + pl * xpl);
        const uintx4 v = {p[0], p[1], p[2], p[3]};
        b = __builtin_bit_cast(bf16x8, v);
    };
    auto mma = [&](floatx16 (&sum)[MK], const OpA &a, const bf16x8 &b) __attribute__((always_inline)) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) sum[mk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mk], b, sum[mk], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    const int NS = P.NO >> 1;
    auto wrap = [&](int at) __attribute__((always_inline)) { return (int)min((unsigned)at, (unsigned)(at - RCB)); };
    int col = 0;
    // operands of step `s` of the unit in buffer b
    auto begin = [&](int b) __attribute__((always_inline)) {
        col = wrap(ring + rcol);
        ya = ybuf + b * YB + aoff;
    };
    auto octet = [&](int s) __attribute__((always_inline)) {
        const int c0 = __builtin_amdgcn_readlane(oct_col, 2 * s), c1 = __builtin_amdgcn_readlane(oct_col, 2 * s + 1);
        const int a0 = __builtin_amdgcn_readlane(oct_at, 2 * s), a1 = __builtin_amdgcn_readlane(oct_at, 2 * s + 1);
        xa = xbuf + (roff + wrap(col + (half ? c1 : c0)) + (half ? a1 : a0));
    };
    auto prime = [&]() __attribute__((always_inline)) {
        // in the order of `step`
        load_b(bl, 2); load_a(ah, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_b(bm, 1); load_a(am, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_b(bh, 0); load_a(al, 2);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto step = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        mma(sum16, ah, bl);
        load_b(bl, 2);
        mma(sum8, ah, bm);
        mma(acc, ah, bh);
        load_a(ah, 0);
        mma(sum16, am, bm);
        load_b(bm, 1);
        mma(sum8, am, bh);
        load_a(am, 1);
        mma(sum16, al, bh);
        load_b(bh, 0);
        load_a(al, 2);
    };
    auto whole_sum = [&](int mk, int v) __attribute__((always_inline)) {
        return fmaf(fmaf(sum16[mk][v], 0x1p-8f, sum8[mk][v]), 0x1p-8f, acc[mk][v]);
    };
    // a tile that this block computed alone; a lane holds one coefficient of 16 filters of each of its MK x 32
    auto store_tile = [&]() __attribute__((always_inline)) {
        const int klim = min(P.Kg - c_kt * TK, TK), r = c_rt * TR + wr * 32 + l32;
        const float rb = rbias && r < P.R ? rbias[r] : 0.f;
        bool odd = false;
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int kl = (wk * MK + mk) * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
                if (kl >= klim || r >= P.R) continue;
                const float val = whole_sum(mk, v);
                odd |= not_finite(val);
                out[(size_t)(c_g * P.Kg + c_kt * TK + kl) * P.R + r] = not_finite(val) ? __uint_as_float(0x7fc00000u) : P.relu ? fmaxf(val + rb, 0.f) : val + rb;
            }
        if (!__any(odd)) return;
        // The wave sums again what is not finite of its part: 14x14x512, 5x5x512x512, 32 images (0.5 ms), one NaN in x 2.9 ms at most, one inf 5.6 (9.0
        // and 17.7 with a result a lane).
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);         // this wave reads back what it stored
#pragma unroll 1
        for (int e = 0; e < MK * 16; ++e) {
            const int kl = (wk * MK + e / 16) * 32 + (e % 16 >> 2) * 8 + half * 4 + (e & 3), k = c_kt * TK + kl;
            const bool there = kl < klim && r < P.R;
            float *o = out + (there ? (size_t)(c_g * P.Kg + k) * P.R + r : 0);
            const bool again = there && not_finite(*(volatile float *)o);
            if (!__any(again)) continue;
            const float val = wave_sum_again(P, x, dzdy, c_g, k, r, again) + rb;
            if (again) *o = P.relu ? fmaxf(val, 0.f) : val;
        }
    };
    auto store_partial = [&](int slot) __attribute__((always_inline)) {
        float *dst = part + (size_t)slot * (TK * TR) + wr * 32 + l32;
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int v = 0; v < 16; ++v) dst[((wk * MK + mk) * 32 + (v >> 2) * 8 + half * 4 + (v & 3)) * TR] = whole_sum(mk, v);
    };
    bool first_segment = true;
    for (int it = 0; it < nunits;) {
        // one segment: the units of one tile in a row
        const int m = min(NU - uu, nunits - it);
        set_tile(t);
        int jc = uu % P.CC;
        auto enter = [&](int u, int i) __attribute__((always_inline)) {
            // the ring: behind the columns of the unit before, or `step` columns on from them
            if (i > 0) ring += 4 * (u == 0 || jc == 0 ? P.SC : P.step) * P.COLP;
            if (ring >= RCB) ring -= RCB;
            if (++jc == P.CC) jc = 0;
            begin(i & 1);
            octet(0);
        };
        await(written + (it & 1), ((it >> 1) + 1) * WGS_STAGE_WAVES);
        enter(0, it);
        prime();
        for (int u = 0; u < m; ++u, ++it) {
            for (int s = 1; s < NS; ++s) {
                ya += 96;
                octet(s);
                step();
            }
            // every operand of this unit is in registers or on its way there
            count(read + (it & 1));
            if (u + 1 < m) {
                await(written + ((it + 1) & 1), (((it + 1) >> 1) + 1) * WGS_STAGE_WAVES);
                enter(u + 1, it + 1);
            }
            step();                    // the segment's last one reads something again, for nothing
        }
        asm volatile("" ::"v"(bh), "v"(bm), "v"(bl), "v"(ah[0]), "v"(am[0]), "v"(al[0]), "v"(ah[MK - 1]), "v"(am[MK - 1]), "v"(al[MK - 1]));
        if (m == NU) store_tile();
        else store_partial(2 * vb + (first_segment ? 0 : 1));
        first_segment = false;
        ++t; uu = 0;
    }
}

}  // namespace mcn
