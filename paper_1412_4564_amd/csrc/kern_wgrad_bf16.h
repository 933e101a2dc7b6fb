// Filter derivative on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16), operands rounded to bf16 (round to nearest even) on chip, fp32
// accumulation: MatConvNet manual (arXiv 1412.4564) Sec. 6.1, dz/dF = phi(x)^T dz/dY summed over the batch, vertical stride 1.
//
// GEMM view, octets (4 rows of one column in 2 images, a pair of images one 32-bit word), slab, ring and units are those of
// kern_wgrad_split.h, with one plane in the place of three:
//   dzdy tile  [filter][octet] in 16-byte words
//   x slab     [channel][image pair][column][row] in 32-bit words
// Eight computing waves of 64 filters x 32*MR coefficients, four waves that fetch and convert, one unit ahead.
//
// What bounds it: what the compute units take in.  A product costs a sixth of the three-plane kernel's, so a staged sample has to meet as
// many filters and coefficients as the accumulators hold (MR up to 3), and a unit takes as long as the staging waves' instructions, some
// 950 of them when they were those of kern_wgrad_split.h (56x56x256, 3x3x256x256, 32 images: 250 us; without products, loads and LDS
// writes still 180).  Hence
//  * x comes by 16-byte loads as dzdy does: a quad of the slab is one in memory.  Rows above the plane are whole quads (XL), rows below it are
//    zeroed as they are packed;
//  * what stays the same along a sweep is worked out where it begins, a unit's columns move the arrays' bases (scalar), and the parameters
//    that only a new sweep needs are read from the kernel's arguments again: 320 instructions for ten octets a thread (190 us);
//  * units of whole columns where LDS and registers allow it: runs of 224 bytes instead of 48 (156 us; 224x224x64, 3x3x64x64, 32 images: units of
//    16 rows 420 us, of 56 rows 213; wgb_us takes 32 rows of two columns for that layer, an estimate of 179.5 against 180.9, and they take 290).
// The kernel before it held eight rows of one image in an octet and the slab Hf times: 335 us and 632 us for the two layers.  It was the faster
// one for 26 of 2000 random layers of 1 to 200 GFLOP by more than 5 %, for ten by more than 20 % (half of them single images, whose octets
// are half empty here); over all of them 193 ms then, 128 now.
//
// A sum that is NaN may be so because a zero in the place of a sample that there is not met an infinity, and is formed again
// (kern_wgrad_split.h); one that is infinite has met no such product and stays.  (Infinite sums formed again too: one infinity in x, 27x27x96,
// 5x5x48x256 in two groups, 128 images, 1.9 ms where an ordinary call takes 0.1.)
//
// Schedules, tiles and the fix-up pass: kern_wgrad.h.
#pragma once
#include "kern_wgrad_split.h"

namespace mcn {

struct WgradBf16Params : WgradSplitParams {
    Div32 dNO, dTIQ, dMC, dT, dHf, dCC, dRB, dTiles, dKT, dRT;
};

// YT, XT: octets of dzdy and of new slab columns that a staging thread brings per unit, at most.
// LINEAR: 1x1 filters, no row of x but those of dzdy is met (no padding, no more output rows than input rows).
// FAR: a unit's images do not fit 31-bit offsets together, one pair of them (NP = 1) with a base for each image does; two more scalars for each
// array, which took 2 % of the time where nothing needs them.
template <int WK, int WR, int MK, int MR, int YT, int XT, bool LINEAR, bool FAR>
__global__ __launch_bounds__(64 * (WK * WR + WGS_STAGE_WAVES), 3) void wgrad_bf16_kernel(WgradBf16Params P, const float *__restrict__ x,
                                                                                      const float *__restrict__ dzdy, float *out,
                                                                                      float *__restrict__ part) {
    constexpr int NT = 64 * WK * WR;               // computing threads
    constexpr int NL = 64 * WGS_STAGE_WAVES;       // staging threads
    constexpr int TK = WK * MK * 32, TR = WR * MR * 32;
    const int NU = P.NU;
    const int T = P.Hf * P.Wf;
    const int YB = (TK * P.PYW + 1) * 16;                // bytes per buffer of dzdy

    extern __shared__ __align__(16) float lds[];
    char *const ybuf = reinterpret_cast<char *>(lds), *const xbuf = ybuf + 2 * YB;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int vb, t, uu, nunits;           // the block's range: nunits units from unit uu of tile t on
    if (P.nchunks > 0) {
        vb = wg_chunk_virtual_block(blockIdx.x, gridDim.x);
        if (vb >= P.nblocks) return;
        const int chunk = div32(vb, P.dTiles);
        t = vb - chunk * P.tiles;
        uu = (int)sk_begin(P.walk, chunk);
        nunits = (int)sk_begin(P.walk, chunk + 1) - uu;
    } else {
        vb = sk_virtual_block(blockIdx.x, P.nblocks);
        const long long ub = sk_begin(P.walk, vb);
        nunits = (int)(sk_begin(P.walk, vb + 1) - ub);
        t = sk_tile(P.walk, ub, NU);
        uu = (int)(ub - (long long)t * NU);
    }
    if (nunits <= 0) return;

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
    // Units follow one another along the columns of a block of rows ("sweep"), so that a unit shares its first columns (all but `step`) with
    // the one before it; they stay where they are, in a ring of RC columns.
    const int first = P.SC - P.step;               // a sweep's first columns
    const int colB = 4 * P.COLP, RCB = colB * P.RC;       // column and ring in bytes

    if (wave >= WK * WR) {
        // ---- the waves that fetch and convert -------------------------------------------------
        // One wave to a SIMD, which a unit takes as long as its instructions: whatever stays the same along a sweep is worked out where one
        // begins, the columns of a unit move the arrays' bases (scalar), and no branch stands between the requests, so that the waits for
        // a word leave the younger ones on their way.
        typedef float Row4 __attribute__((ext_vector_type(4)));          // four rows of an image
        const int ltid = tid - NT;
        // dzdy words (filter, line, quad), quads fastest: column, image pair, row and filter, a byte each; slab words (column, channel, image
        // pair, quad) of a unit's last `step` columns: column, image pair, first row and channel (8, 2, 12, 10 bits)
        unsigned y_at[YT], x_at[XT];
        int y_lds[YT], x_lds[XT];
        auto x_row = [](unsigned at) __attribute__((always_inline)) { return (int)(at >> 10 & 0xfff); };
        constexpr unsigned ABSENT = 0xffffffffu;
#pragma unroll
        for (int s = 0; s < YT; ++s) {
            const int q = ltid + NL * s, k = div32(q, P.dNO), o = q - k * P.NO, line = div32(o, P.dTIQ), m = div32(line, P.dMC), row = 4 * (o - line * P.TIQ), col = line - m * P.MC;
            y_at[s] = q < P.YW ? (unsigned)(col << 24 | m << 16 | row << 8 | k) : ABSENT;
            y_lds[s] = (q < P.YW ? k * P.PYW + o : TK * P.PYW) * 16;
        }
        struct Word { int col, c, m, row, lds; };
        // What is needed once a sweep is read from the kernel's arguments there: kept in scalar registers beside the rest, it went through
        // vector registers (a hundred scalars did)
        typedef const __attribute__((address_space(4))) WgradBf16Params Args;
        auto args = []() __attribute__((always_inline)) {
            Args *a = (Args *)__builtin_amdgcn_kernarg_segment_ptr();
            asm volatile("" : "+s"(a));
            return a;
        };
        auto slab_word = [&](const auto &P, int q) __attribute__((always_inline)) {
            Word w;
            w.col = div32(q, Div32{P.dXW1.m, P.dXW1.l}); q -= w.col * P.XW1;
            const int a = div32(q, Div32{P.dXQ.m, P.dXQ.l});
            w.row = 4 * (q - a * P.XQ);
            w.c = div32(a, Div32{P.dNP.m, P.dNP.l});
            w.m = a - w.c * P.NP;
            w.lds = 4 * (w.c * P.CHP + w.m * P.MPP + w.row);
            return w;
        };
        const int XW = P.step * P.XW1;
#pragma unroll
        for (int s = 0; s < XT; ++s) {
            const int q = ltid + NL * s;
            const Word w = slab_word(P, q);
            x_at[s] = q < XW ? (unsigned)(w.col << 24 | w.m << 22 | w.row << 10 | w.c) : ABSENT;
            x_lds[s] = w.lds + w.col * colB;
        }
        // The unit to request: where it is, and where the arrays' bases are (its first row and column; x: the first row of the slab and the first
        // column that the unit adds; of a pair's first image), with the bytes behind them (FAR: of either image)
        int klim = 0, nch = 0, xch = 0, ych = 0;
        int jr = div32(uu, P.dCC), jc = uu - jr * P.CC, ib = div32(jr, P.dRB), rb = jr - ib * P.RB;
        bool new_tile = true, start = true;                 // start: it shares no column with the one before
        const char *xp = nullptr, *yp = nullptr;
        bool moved = false;                // the bases are those of the sweep
        const int xdown = 4 * (P.TI - P.CC * P.MC * P.Sw * P.xsj), ydown = 4 * (P.TI - P.CC * P.MC * P.ysj);       // from behind a sweep to the next block of rows
        int xleft[FAR ? 2 : 1] = {}, yleft[FAR ? 2 : 1] = {}, rows = 0, below = 0;        // below: rows that the plane has from the slab's first one on
        unsigned vy[YT], vx[XT];           // byte offsets of the words, or out of range (images past the last one lie behind the array)
        auto set_tile = [&](int tt) __attribute__((always_inline)) {
            const int q = div32(tt, P.dRT), rt = tt - q * P.RT, g = div32(q, P.dKT), kt = q - g * P.KT;
            const int r_lo = rt * TR, r_hi = min(r_lo + TR, P.R), c_lo = div32(r_lo, P.dT);
            nch = div32(r_hi - 1, P.dT) - c_lo + 1;
            klim = min(P.Kg - kt * TK, TK);
            xch = g * P.Cg + c_lo;
            ych = g * P.Kg + kt * TK;
            new_tile = true;
        };
        // FAR: below zero where the image is not there, so that a sweep's first columns, at lower addresses, are found absent too
        auto bytes_left = [&](long long elements) __attribute__((always_inline)) {
            constexpr long long LEAST = FAR ? -0x10000000 : 0;
            return elements > 0x1fffffff ? 0x7fffffff : (int)(4 * max(elements, LEAST));
        };
        auto left_of = [&](const int (&left)[FAR ? 2 : 1], int sn, int i) __attribute__((always_inline)) { return FAR ? left[FAR ? i : 0] : left[0] - i * 4 * sn; };
        auto move = [&](int xby, int yby) __attribute__((always_inline)) {
            xp += xby; yp += yby;
#pragma unroll
            for (int i = 0; i < (FAR ? 2 : 1); ++i) { xleft[i] -= xby; yleft[i] -= yby; }
        };
        auto words_there = [&]() __attribute__((always_inline)) {
            Args &P = *args();
#pragma unroll
            for (int s = 0; s < YT; ++s) {
                const int k = y_at[s] & 255, row = y_at[s] >> 8 & 255, m = y_at[s] >> 16 & 255, col = y_at[s] >> 24;
                vy[s] = ((k < klim) & (LINEAR | (row < rows))) ? 4u * ((unsigned)k * P.ysc + (unsigned)col * P.ysj + row + 2u * m * P.ysn) : SLAB_INVALID;
            }
#pragma unroll
            for (int s = 0; s < XT; ++s) {
                const int c = x_at[s] & 0x3ff, row = x_row(x_at[s]), m = x_at[s] >> 22 & 3, col = x_at[s] >> 24;
                // a word begins on a row of the plane or lies wholly above or below it (plan_wgrad_split_shape)
                const bool ok = (c < nch) & (x_at[s] != ABSENT) & (LINEAR | ((unsigned)(row - (below - P.H)) < (unsigned)P.H));
                vx[s] = ok ? 4u * ((unsigned)c * P.xsc + (unsigned)col * P.xsj + row + 2u * m * P.xsn) : SLAB_INVALID;
            }
        };
        auto set_sweep = [&]() __attribute__((always_inline)) {
            const int was_rows = rows, was_below = below;
            rows = min(P.TI, P.Ho - rb * P.TI);
            below = P.H + P.XL - rb * P.TI;
            if (!moved) {
                Args &P = *args();
                const int io0 = rb * P.TI, jo0 = jc * P.MC, n0 = ib * 2 * P.NP;
                const long long xb = (long long)n0 * P.xsn + (long long)xch * P.xsc + (long long)(jo0 * P.Sw - P.Pl + first) * P.xsj + (io0 - P.XL);
                const long long yb = (long long)n0 * P.ysn + (long long)ych * P.ysc + (long long)jo0 * P.ysj + io0;
                // bytes: limited where the sweep's first column would begin, to which the next block of rows goes back
                const int xon = jo0 * P.Sw * P.xsj, yon = jo0 * P.ysj;
                xp = reinterpret_cast<const char *>(x) + 4 * xb;
                yp = reinterpret_cast<const char *>(dzdy) + 4 * yb;
#pragma unroll
                for (int i = 0; i < (FAR ? 2 : 1); ++i) {
                    xleft[i] = bytes_left(P.xtot - (xb - xon) - i * P.xsn) - 4 * xon;
                    yleft[i] = bytes_left(P.ytot - (yb - yon) - i * P.ysn) - 4 * yon;
                }
            }
            moved = false;
            // The words' offsets are those of the sweep before if the same rows of them are there.  LINEAR: rows that are not there meet rows of
            // dzdy that are zeroed.
            auto inside = [&](int at) __attribute__((always_inline)) { return (at <= P.H) & (at >= 4 * P.XQ); };
            if (!new_tile & (LINEAR | ((rows == was_rows) & ((below == was_below) | (inside(below) & inside(was_below)))))) return;
            new_tile = false;
            words_there();
        };
        // four pairs of samples, a pair of images each; of rows that there are not, `end` and on, zeros
        auto pack = [&](Row4 a, Row4 b) __attribute__((always_inline)) { return uintx4{pack_bf16x2(a[0], b[0]), pack_bf16x2(a[1], b[1]), pack_bf16x2(a[2], b[2]), pack_bf16x2(a[3], b[3])}; };
        auto pack_rows = [&](Row4 a, Row4 b, int row, int end) __attribute__((always_inline)) {
            uintx4 w = pack(a, b);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = row < end - e ? w[e] : 0;
            return w;
        };
        auto put_x = [&](const Row4 (&v)[2], int row, int end, int at, bool there) __attribute__((always_inline)) {
            const uintx4 w = LINEAR ? pack(v[0], v[1]) : pack_rows(v[0], v[1], row, end);
            if (there) {
                unsigned *dst = reinterpret_cast<unsigned *>(xbuf + at);
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[e] = w[e];
            }
        };
        auto load = [&](__amdgpu_buffer_rsrc_t rs, unsigned off) __attribute__((always_inline)) { return __builtin_bit_cast(Row4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0)); };
        // What is on its way: one unit, every word of it requested as soon as the same word of the unit before has been written, so
        // that it has a unit's time to come.
        Row4 yv[YT][2], xv[XT][2];
        bool c_start = false;              // of that unit
        int c_rows = 0, c_below = 0, c_nch = 0, c_j0 = 0, c_xleft[FAR ? 2 : 1] = {};
        const char *c_xp = nullptr;
        int ring = first;                  // the column of the ring where those that it adds begin
        // A sweep's first unit: the columns that a unit otherwise finds in place.  Requested and written here, while the unit before is computed: held
        // in registers until then they would leave none for units of this size.
        auto first_columns = [&]() __attribute__((always_inline)) {
            Args &P = *args();
            const int extra = first * P.XW1, back = 4 * first * P.xsj;       // words; bytes from them to the columns that the unit adds
#pragma unroll 1
            for (int q0 = ltid; q0 - ltid < extra; q0 += 2 * NL) {
                Row4 v[2][2];
                Word w[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int q = q0 + NL * s;
                    w[s] = slab_word(P, q);
                    const bool ok = (q < extra) & (w[s].c < c_nch) & ((unsigned)(c_j0 + w[s].col) < (unsigned)P.W) & ((unsigned)(w[s].row - (c_below - P.H)) < (unsigned)P.H);
                    const unsigned off = ok ? 4u * ((unsigned)w[s].c * P.xsc + (unsigned)w[s].col * P.xsj + w[s].row + 2u * w[s].m * P.xsn) : SLAB_INVALID;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        v[s][i] = load(__builtin_amdgcn_make_buffer_rsrc((void *)(c_xp + 4ll * i * P.xsn - back), 0, max(c_xleft[FAR ? i : 0] > 0x7fffffff - back ? 0x7fffffff : left_of(c_xleft, P.xsn, i) + back, 0), BUFFER_FLAGS), off);
                }
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const int at = ring - first + w[s].col;
                    put_x(v[s], w[s].row, c_below, w[s].lds + (at < 0 ? at + P.RC : at) * colB, q0 + NL * s < extra);
                }
            }
        };
        // put: the unit on its way into the buffers b; get: request the next one
        auto stage = [&](int b, auto put, auto get) __attribute__((always_inline)) {
            if constexpr (!LINEAR)
                if (put && c_start && first > 0) first_columns();
            if (get && start) set_sweep();
            __amdgpu_buffer_rsrc_t yrs[2], xrs[2];         // of a pair's images
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                yrs[i] = __builtin_amdgcn_make_buffer_rsrc((void *)(yp + 4ll * i * P.ysn), 0, max(left_of(yleft, P.ysn, i), 0), BUFFER_FLAGS);
                xrs[i] = __builtin_amdgcn_make_buffer_rsrc((void *)(xp + 4ll * i * P.xsn), 0, max(left_of(xleft, P.xsn, i), 0), BUFFER_FLAGS);
            }
            const unsigned ycols = (unsigned)min(max(P.Wo - jc * P.MC, 0), 255) << 24;
            const int j0 = jc * P.MC * P.Sw - P.Pl + first, xlo = min(max(-j0, 0), 255), xhi = min(max(P.W - j0, xlo), 255);
            const unsigned xfrom = (unsigned)xlo << 24, xcols = (unsigned)(xhi - xlo) << 24;
            const int ybuf_b = b * YB, to = ring * colB;
            const unsigned room = (unsigned)min(P.RC - ring, 255) << 24;          // columns up to the ring's end
#pragma unroll
            for (int s = 0; s < YT; ++s) {
                if (put) {
                    // rows past the patch's last one are those of the next column: they must not count
                    *reinterpret_cast<uintx4 *>(ybuf + ybuf_b + y_lds[s]) = pack_rows(yv[s][0], yv[s][1], y_at[s] >> 8 & 255, c_rows);
                }
                if (get) {
                    const unsigned off = y_at[s] < ycols ? vy[s] : SLAB_INVALID;
#pragma unroll
                    for (int i = 0; i < 2; ++i) yv[s][i] = load(yrs[i], off);
                }
                // requests in one order wherever they are made: the waits for a word have to hold for all of them
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int s = 0; s < XT; ++s) {
                if (put) put_x(xv[s], x_row(x_at[s]), c_below, x_lds[s] + (x_at[s] < room ? to : to - RCB), x_at[s] != ABSENT);
                if (get) {
                    const unsigned off = x_at[s] - xfrom < xcols ? vx[s] : SLAB_INVALID;
#pragma unroll
                    for (int i = 0; i < 2; ++i) xv[s][i] = load(xrs[i], off);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (get) {
                if (put) {
                    ring += start ? first + P.step : P.step;
                    if (ring >= P.RC) ring -= P.RC;
                }
                c_start = start; c_rows = LINEAR ? min(P.TI, P.Ho - rb * P.TI) : rows; c_below = below;
                if constexpr (!LINEAR) {
                    c_nch = nch; c_j0 = j0 - first; c_xp = xp;
#pragma unroll
                    for (int i = 0; i < (FAR ? 2 : 1); ++i) c_xleft[i] = xleft[i];
                }
                start = false;
                move(4 * P.MC * P.Sw * P.xsj, 4 * P.MC * P.ysj);
                if (++jc == P.CC) {
                    jc = 0; start = !LINEAR; moved = true;
                    move(xdown, ydown);
                    if (++rb == P.RB) {
                        rb = 0; moved = false; start = true;
                        if (++ib == P.IB) { ib = 0; if (++t < P.tiles) set_tile(t); }
                    }
                }
            }
        };
        struct Yes { __device__ constexpr operator bool() const { return true; } };
        struct No { __device__ constexpr operator bool() const { return false; } };
        set_tile(t);
        stage(0, No(), Yes());
        int it = 0;
        for (; it + 1 < nunits; ++it) {        // unit it is written while unit it - 1 is computed
            await(read + (it & 1), (it >> 1) * (WK * WR));
            stage(it & 1, Yes(), Yes());
            count(written + (it & 1));
        }
        await(read + (it & 1), (it >> 1) * (WK * WR));
        stage(it & 1, Yes(), No());
        count(written + (it & 1));
        return;
    }

    // ---- the computing waves -------------------------------------------------------------------
    const int wk = wave % WK, wr = wave / WK;
    floatx16 sum[MK][MR];
    int c_rt = 0, c_kt = 0, c_g = 0, roff[MR], rcol[MR];      // roff, rcol: where the lane's coefficients are in the slab, in bytes, but for the column; their columns
    auto set_tile = [&](int tt) __attribute__((always_inline)) {
        const int q = div32(tt, P.dRT);
        c_rt = tt - q * P.RT;
        c_g = div32(q, P.dKT); c_kt = q - c_g * P.KT;
        const int c_lo = div32(c_rt * TR, P.dT);
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) {
            const int r = c_rt * TR + (wr * MR + mr) * 32 + l32;
            roff[mr] = rcol[mr] = 0;
            if (r < P.R) {
                const int c = div32(r, P.dT), tap = r - c * T, fj = div32(tap, P.dHf);
                roff[mr] = 4 * ((c - c_lo) * P.CHP + tap - fj * P.Hf + P.XL - P.Pt);
                rcol[mr] = fj * colB;
            }
        }
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int mr = 0; mr < MR; ++mr)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[mk][mr][v] = 0.f;
    };
    // Lane o: where octet o of a unit starts in the slab, in bytes: its column and the rest apart.  An octet is (line, rows 4*q on),
    // line = (image pair, column).  Read across lanes: a table in LDS would make every step wait for all of its operands.
    int oct_col, oct_at;
    {
        const int line = div32(lane, P.dTIQ), q = lane - line * P.TIQ, m = div32(line, P.dMC), dc = line - m * P.MC;
        oct_col = dc * P.Sw * colB;
        oct_at = 4 * (m * P.MPP + 4 * q);
    }
    bf16x8 oa[MK], ob[MR];
    const int aoff = ((wk * MK * 32 + l32) * P.PYW + half) * 16, amk = 32 * P.PYW * 16;
    const char *ya = ybuf;            // the lane's octets of the next operands
    const char *xa[MR];
    int ring = 0;                     // the unit's first column, in bytes
    auto load_a = [&](int mk) __attribute__((always_inline)) { oa[mk] = *reinterpret_cast<const bf16x8 *>(ya + mk * amk); };
    auto load_b = [&](int mr) __attribute__((always_inline)) {
        const unsigned *p = reinterpret_cast<const unsigned *>(xa[mr]);
        const uintx4 v = {p[0], p[1], p[2], p[3]};
        ob[mr] = __builtin_bit_cast(bf16x8, v);
    };
    auto mma = [&](int mk, int mr) __attribute__((always_inline)) {
        sum[mk][mr] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(oa[mk], ob[mr], sum[mk][mr], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    const int NS = P.NO >> 1;
    auto wrap = [&](int at) __attribute__((always_inline)) { return (int)min((unsigned)at, (unsigned)(at - RCB)); };
    int col[MR];
    // operands of step `s` of the unit in buffer b
    auto begin = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) col[mr] = wrap(ring + rcol[mr]);
        ya = ybuf + b * YB + aoff;
    };
    auto octet = [&](int s) __attribute__((always_inline)) {
        const int c0 = __builtin_amdgcn_readlane(oct_col, 2 * s), c1 = __builtin_amdgcn_readlane(oct_col, 2 * s + 1);
        const int a0 = __builtin_amdgcn_readlane(oct_at, 2 * s), a1 = __builtin_amdgcn_readlane(oct_at, 2 * s + 1);
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) xa[mr] = xbuf + (roff[mr] + wrap(col[mr] + (half ? c1 : c0)) + (half ? a1 : a0));
    };
    auto prime = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) load_a(mk);
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) load_b(mr);
        __builtin_amdgcn_sched_barrier(0);
    };
    // every operand is read for the next step as soon as its last product is issued
    auto step = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) {
#pragma unroll
            for (int mk = 0; mk < MK; ++mk) {
                mma(mk, mr);
                if (mr == MR - 1) load_a(mk);
            }
            load_b(mr);
        }
    };
    // a tile that this block computed alone; a lane holds one coefficient of 16 filters of each of its MK x MR x 32
    auto store_tile = [&]() __attribute__((always_inline)) {
        const int klim = min(P.Kg - c_kt * TK, TK), r0 = c_rt * TR + wr * MR * 32 + l32;
        bool odd = false;
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) {
            const int r = r0 + mr * 32;
#pragma unroll
            for (int mk = 0; mk < MK; ++mk)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int kl = (wk * MK + mk) * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
                    if (kl >= klim || r >= P.R) continue;
                    const float val = sum[mk][mr][v];
                    odd |= val != val;
                    out[(size_t)(c_g * P.Kg + c_kt * TK + kl) * P.R + r] = val;
                }
        }
        if (!__any(odd)) return;
        // the wave sums again what is NaN of its part, from the operands as they are
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);         // this wave reads back what it stored
#pragma unroll 1
        for (int e = 0; e < MK * MR * 16; ++e) {
            const int mr = e / (MK * 16), r = r0 + mr * 32, kl = (wk * MK + e / 16 - mr * MK) * 32 + (e % 16 >> 2) * 8 + half * 4 + (e & 3), k = c_kt * TK + kl;
            const bool there = kl < klim && r < P.R;
            float *o = out + (there ? (size_t)(c_g * P.Kg + k) * P.R + r : 0);
            const float was = there ? *(volatile float *)o : 0.f;
            const bool again = was != was;
            if (!__any(again)) continue;
            const float val = wave_sum_again(P, x, dzdy, c_g, k, r, again);
            if (again) *o = val;
        }
    };
    auto store_partial = [&](int slot) __attribute__((always_inline)) {
        float *dst = part + (size_t)slot * (TK * TR) + wr * MR * 32 + l32;
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int mr = 0; mr < MR; ++mr)
#pragma unroll
                for (int v = 0; v < 16; ++v) dst[((wk * MK + mk) * 32 + (v >> 2) * 8 + half * 4 + (v & 3)) * TR + mr * 32] = sum[mk][mr][v];
    };
    bool first_segment = true;
    for (int it = 0; it < nunits;) {
        // one segment: the units of one tile in a row
        const int m = min(NU - uu, nunits - it);
        set_tile(t);
        int jc = uu - div32(uu, P.dCC) * P.CC;
        auto enter = [&](int u, int i) __attribute__((always_inline)) {
            // the ring: `step` columns on from the unit before, and behind its columns where it is another sweep's
            if (i > 0) ring += (u == 0 || jc == 0 ? P.SC : P.step) * colB;
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
                ya += 32;
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
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) asm volatile("" ::"v"(oa[mk]));
#pragma unroll
        for (int mr = 0; mr < MR; ++mr) asm volatile("" ::"v"(ob[mr]));
        if (m == NU) store_tile();
        else store_partial(2 * vb + (first_segment ? 0 : 1));
        first_segment = false;
        ++t; uu = 0;
    }
}

}  // namespace mcn
