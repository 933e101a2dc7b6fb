// Implicit-GEMM convolution of fp32 operands on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16).
//
// The sum is that of kern_igemm.h (MatConvNet manual, arXiv 1412.4564, Sec. 4.1), in fp32 precision: every operand v is
// held on chip as three bf16 planes, v = hi + mid / 2^8 + lo / 2^16 exactly (split_bf16x3), and a product is formed as
//   w_hi*x_hi + (w_hi*x_mid + w_mid*x_hi) / 2^8 + (w_mid*x_mid + w_lo*x_hi + w_hi*x_lo) / 2^16
// with fp32 accumulation.  Each product of two bf16 numbers is exact in fp32 and what is left out (w_mid*x_lo and
// smaller) is below 2^-26 of |w||x|, less than the rounding of one fp32 multiply-add.  The three scales have accumulators of
// their own, put together at the end: the planes can then carry operands of every size (split_bf16x3), and an MFMA rounds its
// sum four times on the way through its 16 elements: with all six products in one sum the results are 1.2 times as far from
// sums in 64 bits as those of the fp32 instructions (24 roundings per 16 elements against 16); the roundings of the scaled
// sums cost nothing.  Six products on a matrix core that multiplies 16 times as fast as in fp32 cost 6/16 of the fp32 kernel's
// matrix time.
//
// Tiling, pixel numbering, schedule and fix-up pass: kern_igemm.h.  One MFMA takes 16 channels of one tap, a lane's operand
// is 16 consecutive bytes: slab [plane][octet][column][row][8 channels] in LDS, weights
// [channel group][tap][plane][octet][filter][8 channels] in memory (igemm_pack_weights_bf16_kernel, three planes).  A unit
// is 16 channels x all taps, of 1x1 filters several groups of 16 channels (GROUPED).
//
// What bounds it: the matrix core, at the clock that its power leaves, and the waits between its products (two groups of 5x5, 128
// images: 0.68 to 0.73 of the active cycles execute products, at 1.86 GHz of 2.4; a loop of products alone reaches 1.85 PFLOP/s on
// random data and 2.45 on zeros, this kernel 1.3).  Hence
//  * the weights go from the L2 straight into the registers of the waves that use them (waves of one block read the same
//    ones through the L1: 32 bytes a cycle) and not through LDS: staged there, 12 KB per tap, they forced a barrier every
//    tap or two, and with eight waves in step the scalar work, the LDS latency and the skew at each barrier cost as much
//    as half a tap's MFMAs (27x27x96 plane, 5x5x48x256 filters, 128 images: 318 us, now 262, 1.31 PFLOP/s of bf16
//    products; the fp32 kernel 440).  The LDS then holds three slabs and its reads are halved.
//  * slabs are published one barrier before they are computed, so the last step of a unit reads the next unit's first
//    operands and no wave starts a unit with empty registers.
//  * every plane has one set of registers, read anew for the next step as soon as its last product is issued; the order
//    of the products leaves 3 to 5 products (weights) or 2 to 5 (pixels), of MK*MP MFMAs each, between that and the next use.
//
// Row pairs (template flag F23): 3x3 filters at stride 1 through the identity F(2,3) of kern_igemm.h, two thirds of the
// MFMAs.  A "pixel" is a pair of output rows.  Each of the four sums m0..m3 is a convolution of its own with a filter of
// three columns and one row, of a row combination of the input (d0-d2, d1+d2, d2-d1, d1-d3, formed in fp32 before the
// split) with a row combination of the weights, so the waves compute them one after the other with one set of
// accumulators, and add each unit's to the pair's two rows (y0 += m0 + m1 + m2, y1 += m1 - m2 - m3): the sums that the
// MFMAs round are short.  A unit is 16 channels of one combination, the four of a group follow one another.
// Three sums and two rows a result: registers for tiles of 128 filters x 64 pairs, on four computing waves (one a SIMD; eight waves of
// half as much each take 1 to 3 % longer), which hold the weights of a whole unit.
// It takes fewer MFMAs than the other kernel and more staging (two loads per pair, combination and column for three taps,
// against one per pixel for nine), and that bounds it on all but planes too small to fill the chip's tiles, where the
// split of the reduction counts: 14x14x512, 3x3x512x512: 32 images 195 -> 173 us, one image 57 -> 39 us against the fp32
// row-pair kernel (split_pairs_possible in igemm_plan.h; on tiles of 128 pairs, with operands held less exactly, 56x56x256, 32 images
// 596 -> 663 us, 224x224x64 663 -> 822 us).
#pragma once
#include "kern_igemm_bf16.h"

namespace mcn {

constexpr int SPLIT_SLABS = 3;         // slab buffers: computed, next (being read ahead), written
constexpr int SPLIT_BIASES = 4;        // bias buffers: a bias is written at most two tiles ahead
constexpr int SPLIT_STAGE_WAVES = 4;   // waves that fetch and split the input
// Slab samples of a unit, at most: a staging thread brings two of them (16 channels, as many registers, in three sets), or, of
// row pairs, half a one (8 channels of two rows each, in two sets; whole ones on half of the threads: 14x14x512, 3x3x512x512, one image
// 39.9 -> 38.7 us, eight images 69 -> 67 us).
__device__ __host__ constexpr int split_samples(bool f23) { return 64 * SPLIT_STAGE_WAVES * (f23 ? 1 : 4) / 2; }

// ---- results that are not finite -------------------------------------------------------
// An operand that is infinite splits into (inf, nan, nan), so every result that it enters comes out as NaN where the plain
// sum may say +-inf (and one within 2^-9 of the largest float rounds to inf in its hi plane).  Results that are not finite
// are summed again as Sec. 4.1 writes them, in fp32, from the arrays in memory.

// The view as such a sum sees it: filter size and stride (those of IgemmParams describe pairs of rows in a view of row
// pairs), and where weight (group g, filter k, channel c, tap (ti, tj)) is in the caller's array:
// wo + g*wg + k*wk + c*wc + ti*wi + tj*wj (merged phases: shape of that array and the largest b0 per direction, see PackParams)
struct PlainView {
    int Hf, Sh, Wf, Sw;
    int wo, wg, wk, wc, wi, wj;
    int HfA, WfA, DfA, B0i, B0j;
};

// NF results: filters k0 .. k0+NF-1 of pixel (io, jo, n) of group g, those whose bit of `need` is set; s: their bias, then the
// sum.  A lane whose results are all NaN is done.  Bound by address arithmetic and latency: the x of a tap and channel is read
// once for all NF filters, the loads of four channels are in flight together.  A diverged batch (NaN) costs little, an infinite
// operand among ordinary ones a fraction of a millisecond, infinite results everywhere ten times the call and more
// (27x27x96, 5x5x48x256 in two groups, 128 images, forward, 0.35 ms: one NaN 0.36 ms, one inf 1.6 ms, all NaN 0.75 ms, +inf
// everywhere 10.7 ms; one result at a time and to the end of its sum 5.2, 5.6, 33.9 and 33.9 ms).
template <int NF, bool MERGED>
__device__ inline void plain_results(const IgemmParams &P, const PlainView &V, const float *in, const float *w, int g, int k0, int io, int jo,
                                     int n, unsigned need, float (&s)[NF]) {
    const size_t HW = (size_t)P.H * P.W, wc = MERGED ? (size_t)V.HfA * V.WfA * V.DfA : (size_t)V.wc;
    const float *const xg = in + HW * (g * P.Cg + (size_t)P.Ctot * n);
    auto more = [&]() __attribute__((always_inline)) {
        bool m = false;
#pragma unroll
        for (int f = 0; f < NF; ++f) m |= (need >> f & 1) && s[f] == s[f];
        return m;
    };
#pragma unroll 1
    for (int tj = 0; tj < V.Wf; ++tj)
#pragma unroll 1
        for (int ti = 0; ti < V.Hf; ++ti) {
            const int xi = V.Sh * io + ti - P.Pt, xj = V.Sw * jo + tj - P.Pl;
            if (xi < 0 || xi >= P.H || xj < 0 || xj >= P.W || !more()) continue;
            const float *xp = xg + xi + (size_t)P.H * xj;
            const float *wp[NF];
            bool tap[NF];                              // merged phases: the filter's phase has this tap
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int k = min(k0 + f, P.Kg - 1);
                tap[f] = true;
                if constexpr (MERGED) {
                    const int ph = k / P.mD, mc = k - ph * P.mD, pj = ph / P.osi, pi = ph - pj * P.osi;
                    const int fi = merged_tap(ti, V.Hf, V.HfA, P.osi, P.mPt, V.B0i, pi), fj = merged_tap(tj, V.Wf, V.WfA, P.osj, P.mPl, V.B0j, pj);
                    tap[f] = fi >= 0 && fj >= 0;
                    wp[f] = w + (tap[f] ? fi + V.HfA * fj : 0) + (size_t)V.HfA * V.WfA * (mc + (size_t)V.DfA * (g * P.Cg));
                } else {
                    wp[f] = w + (V.wo + g * V.wg + k * V.wk + ti * V.wi + tj * V.wj);
                }
            }
#pragma unroll 1
            for (int c0 = 0; c0 < P.Cg; c0 += 4) {
                const bool full = c0 + 4 <= P.Cg;
                float xv[4], wv[4][NF];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const size_t c = full ? c0 + u : min(c0 + u, P.Cg - 1);
                    xv[u] = xp[c * HW];
#pragma unroll
                    for (int f = 0; f < NF; ++f) wv[u][f] = wp[f][c * wc];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const float next = fmaf(wv[u][f], xv[u], s[f]);
                        s[f] = c0 + u < P.Cg && (!MERGED || tap[f]) ? next : s[f];
                    }
                if (!__any(more())) break;
            }
        }
}

// in the fix-up pass: four consecutive pixels from q on, of one filter
struct PlainPixels {
    static constexpr bool on = true;
    PlainView V;
    const float *in, *w;
    __device__ void pixels(const IgemmParams &P, const float *bias, int g, int rb, int kl, int q0, float (&v)[4]) const {
        if (!(not_finite(v[0]) || not_finite(v[1]) || not_finite(v[2]) || not_finite(v[3]))) return;
        const float b = bias ? bias[P.mD ? g * P.mD + kl % P.mD : g * P.Kg + kl] : 0.f;
#pragma unroll 1
        for (int j = 0; j < 4; ++j) {
            const float was = j == 0 ? v[0] : j == 1 ? v[1] : j == 2 ? v[2] : v[3];
            const int q = q0 + j, c = div32(q, P.dTI), n = div32(c, P.dWo), jo = c - n * P.Wo, io = rb * P.TI + q - c * P.TI;
            if (!not_finite(was) || q >= P.QN || io >= P.Ho) continue;
            float s[1] = {b};
            if (P.mD) plain_results<1, true>(P, V, in, w, g, kl, io, jo, n, 1u, s);
            else plain_results<1, false>(P, V, in, w, g, kl, io, jo, n, 1u, s);
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = u == j ? s[0] : v[u];
        }
    }
};

// What the main kernel goes by, and (read from the kernel's arguments in memory, where this is the first one) the repair of
// its tiles.
// Beside IgemmParams, not in it, so that the other kernels' arguments stay where they are (31x31x56, 5x5x56x64, 123 images, a step 1.012 times as long
// with these fields among them, 1.006 without, against before there were any).
struct FoldedChannels {
    // channels of the reduction: Cg, or, of a view whose channels are the stride phases of the input's (folded_view; strides fSh, fSw), Cg*fSh*fSw
    int VC, fSh, fSw;
    Div32 dfSh, dfSS;          // by fSh, by fSh*fSw
};
struct SplitParams : IgemmParams {
    PlainView V;
    FoldedChannels F;
    const float *in, *w, *bias;
    float *out;
};

// A wave's part of a stored tile t: results that are not finite (the ReLU must not hide them: they are stored as NaN) are read
// back, four filters of the lane's pixel at a time, and replaced.  params_lo, params_hi: where the kernel's arguments are in memory.
// What it needs it reads from there anew: taken from the kernel's own copies, with the kernel's sums still alive around it, it
// cost the kernel up to 240 spilled vector registers.
template <int TK, int WK, int MK, int MP, int TQ, int ROWS, bool MERGED>
__device__ __attribute__((always_inline)) inline void repair_tile(unsigned params_lo, unsigned params_hi, int t, int wave) {
    const size_t at = (size_t)(unsigned)__builtin_amdgcn_readfirstlane(params_hi) << 32 | (unsigned)__builtin_amdgcn_readfirstlane(params_lo);
    const SplitParams &P = *(const SplitParams *)(const __attribute__((address_space(4))) void *)at;
    t = __builtin_amdgcn_readfirstlane(t);
    wave = __builtin_amdgcn_readfirstlane(wave);
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), half = lane >> 5, wk = wave % WK, wp = wave / WK;
    int kt, pt, rb, g;
    decode_tile(P, t, &kt, &pt, &rb, &g);
    const int OHW = P.OH * P.OW;
    __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);           // this wave reads back what it stored
#pragma unroll 1
    for (int e = 0; e < MK * MP * ROWS * 4; ++e) {
        const int row = e % ROWS, v4 = e / ROWS % 4, mk = e / (4 * ROWS) % MK, mp = e / (4 * ROWS * MK);
        const int q = pt * TQ + (wp * MP + mp) * 32 + (lane & 31);
        const int c = div32(q, P.dTI);
        const int n = div32(c, P.dWo);
        const int jo = c - n * P.Wo, pair = rb * P.TI + q - c * P.TI, io = ROWS * pair + row;      // io: row of the view
        const bool pixel = q < P.QN && (ROWS == 2 ? io < P.wino_Ho : pair < P.Ho);
        const int k0 = kt * TK + (wk * MK + mk) * 32 + v4 * 8 + half * 4;
        unsigned need = 0;
        float s[4], *o[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            bool there = pixel && k0 + f < P.Kg;
            int oi = P.oi0 + P.osi / ROWS * io, oj = P.oj0 + P.osj * jo, ch = g * P.Kg + k0 + f;
            if constexpr (MERGED) {
                const MergedFilter m = merged_filter(P, k0 + f);
                oi = m.i0 + P.osi * io; oj = m.j0 + P.osj * jo; ch = g * P.mD + m.c;
                there = there && oi < P.OH && oj < P.OW;
            }
            o[f] = P.out + (there ? (size_t)oi + (size_t)P.OH * oj + (size_t)OHW * (ch + (size_t)P.Ktot * n) : 0);
            if (there && not_finite(*(const volatile float *)o[f])) need |= 1u << f;
            s[f] = P.bias && there ? P.bias[ch] : 0.f;
        }
        if (need == 0) continue;
        plain_results<4, MERGED>(P, P.V, P.in, P.w, g, k0, io, jo, n, need, s);
#pragma unroll
        for (int f = 0; f < 4; ++f)
            if (need >> f & 1) *o[f] = P.relu ? fmaxf(s[f], 0.f) : s[f];
    }
}

// Row pairs: as a function, which the kernel's sums, in more registers there, stay clear of (14x14x512, 3x3x512x512, 32 images: 186 us,
// 190 with it inside).  The others keep it inside: a call takes stack in memory, up to 180 bytes a lane for merged phases, which the
// runtime sets aside for every wave that fits the chip (94 MB).
template <int TK, int WK, int MK, int MP, int TQ>
__device__ __attribute__((noinline)) void repair_pairs(unsigned params_lo, unsigned params_hi, int t, int wave) {
    repair_tile<TK, WK, MK, MP, TQ, 2, false>(params_lo, params_hi, t, wave);
}

// Weights for F23: [g][kt][unit][filter column][plane][octet][kk][8 channels]; a thread reads the three rows of one filter
// column for two channels and writes all planes of their four combinations.
__global__ __launch_bounds__(256) void igemm_pack_f23_split_kernel(const float *__restrict__ w, unsigned *__restrict__ packed, PackParams Q) {
    const int NCG = Q.NU / 4;
    int p = blockIdx.x * 256 + threadIdx.x;
    const int j2 = p & 3; p >>= 2;
    const int kk = p % Q.TK; p /= Q.TK;
    const int oct = p & 1; p >>= 1;
    const int fj = p % 3; p /= 3;
    const int cg = p % NCG; p /= NCG;
    const int kt = p % Q.KT;
    const int g = p / Q.KT;
    if (g >= Q.G) return;
    const int k = kt * Q.TK + kk;
    float v[2][4] = {};
    for (int e = 0; e < 2; ++e) {
        const int c = cg * BF_DC + oct * 8 + 2 * j2 + e;
        if (k >= Q.Kg || c >= Q.Cg) continue;
        const float *src = Q.mode == 0 ? w + 3 * (fj + 3 * (c + (size_t)Q.DfA * (g * Q.Kg + k)))
                                       : w + 3 * ((2 - fj) + 3 * (k + (size_t)Q.DfA * (g * Q.Cg + c)));
        const float g0 = Q.mode == 0 ? src[0] : src[2], g1 = src[1], g2 = Q.mode == 0 ? src[2] : src[0];   // dzdx: the flipped filter
        v[e][0] = g0;
        v[e][1] = 0.5f * (g0 + g1 + g2);
        v[e][2] = 0.5f * (g0 - g1 + g2);
        v[e][3] = g2;
    }
    for (int combo = 0; combo < 4; ++combo) {
        const int uu = 4 * cg + combo;
        unsigned *dst = packed + ((size_t)(g * Q.KT + kt) * Q.NU + uu) * Q.WSZ + (fj * 6 + oct) * Q.TK * 4 + kk * 4 + j2;
        unsigned hi, mid, lo;
        split_bf16x3(v[0][combo], v[1][combo], &hi, &mid, &lo);
        dst[0] = hi; dst[2 * Q.TK * 4] = mid; dst[4 * Q.TK * 4] = lo;
    }
}

// The words of igemm_pack_weights_bf16_kernel, or (F23, mode 0 alone) of the one above, where the taps of 16 channels of 16 filters are 16 runs of the caller's
// array (modes 0 and 1 without strides).  A block brings those runs into LDS by 16-byte loads and writes every tap of them from there, a wave the 16
// filters of an octet of channels at a time.  With a pair of weights to a thread, 4 bytes of a line to a load, every tap takes the line
// anew, on whichever XCD its block is.
// Bound by the way of the words through memory where there are many (3x3x512x512 as row pairs, forward: 28 MB, 9.8 -> 7.4 us; two planes 10.5 -> 7.0,
// one 10.7 -> 6.2; 5x5x512x512 in three planes 28 -> 13 us), by the chain from load to store in a block where there are few (pack_run_blocks).
constexpr int PACK_RUN = 16, PACK_RUN_TAPS = 32;
constexpr int pack_run_threads(bool f23) { return f23 ? 384 : 256; }      // row pairs: a wave to a filter column and octet of channels
__device__ __host__ inline int pack_run_pitch(int taps) { return PACK_RUN * taps + 4; }      // keeps 16-byte words whole, and filters off each other's banks
template <int PLANES, bool F23>
__global__ __launch_bounds__(pack_run_threads(F23)) void igemm_pack_runs_kernel(const float *__restrict__ w, unsigned *__restrict__ packed, PackParams Q) {
    static_assert(!F23 || PLANES == 3, "row pairs: three planes");
    typedef float Quad __attribute__((ext_vector_type(4), aligned(4)));
    extern __shared__ __align__(16) float runs[];      // [16 filters (mode 0) or channels (mode 1)][16 of the other][tap]
    const int T = Q.HfA * Q.WfA, pitch = pack_run_pitch(T), per = F23 ? 4 : Q.NTR, NCG = Q.NU / per;
    int t = blockIdx.x;
    const int kk0 = t % (Q.TK / PACK_RUN) * PACK_RUN; t /= Q.TK / PACK_RUN;
    const int cg = t % NCG; t /= NCG;
    const int kt = t % Q.KT, g = t / Q.KT, k0 = kt * Q.TK + kk0, c0 = cg * BF_DC;
    const int filters = min(Q.Kg - k0, PACK_RUN), channels = min(Q.Cg - c0, BF_DC);      // none of them: zeros
    {
        constexpr int LANES = pack_run_threads(F23) / PACK_RUN;       // to a run
        const int r = threadIdx.x / LANES, rows = Q.mode == 0 ? filters : channels, length = r < rows ? T * max(Q.mode == 0 ? channels : filters, 0) : 0;
        const float *src = w + T * (Q.mode == 0 ? c0 + (size_t)Q.DfA * (g * Q.Kg + k0 + r) : k0 + (size_t)Q.DfA * (g * Q.Cg + c0 + r));
#pragma unroll 4
        for (int e = 4 * (threadIdx.x % LANES); e < PACK_RUN * T; e += 4 * LANES) {
            Quad v = {0.f, 0.f, 0.f, 0.f};
            if (e + 4 <= length) v = *reinterpret_cast<const Quad *>(src + e);
            else
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    if (e + u < length) v[u] = src[e + u];
            *reinterpret_cast<float4 *>(runs + r * pitch + e) = float4{v[0], v[1], v[2], v[3]};
        }
    }
    __syncthreads();
    const int j2 = threadIdx.x & 3, kk = (threadIdx.x >> 2) & 15;
    const int k_step = Q.mode == 0 ? pitch : T, c_step = Q.mode == 0 ? T : pitch;
    unsigned *const group = packed + ((size_t)(g * Q.KT + kt) * Q.NU + (size_t)cg * per) * Q.WSZ + (kk0 + kk) * 4 + j2;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto store = [&](unsigned *dst, float v0, float v1) {
        if constexpr (PLANES == 1) {
            dst[0] = pack_bf16x2(v0, v1);
        } else if constexpr (PLANES == 2) {
            unsigned hi, lo;
            split_bf16x2(v0, v1, &hi, &lo);
            dst[0] = hi; dst[2 * Q.TK * 4] = lo;
        } else {
            unsigned hi, mid, lo;
            split_bf16x3(v0, v1, &hi, &mid, &lo);
            dst[0] = hi; dst[2 * Q.TK * 4] = mid; dst[4 * Q.TK * 4] = lo;
        }
    };
    if constexpr (F23) {
        const int oct = wave & 1, fj = wave >> 1;
        float v[2][4];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float *q = runs + kk * k_step + (oct * 8 + 2 * j2 + e) * c_step + 3 * fj;
            const float g0 = q[0], g1 = q[1], g2 = q[2];
            v[e][0] = g0;
            v[e][1] = 0.5f * (g0 + g1 + g2);
            v[e][2] = 0.5f * (g0 - g1 + g2);
            v[e][3] = g2;
        }
#pragma unroll
        for (int combo = 0; combo < 4; ++combo) store(group + (size_t)combo * Q.WSZ + (fj * 6 + oct) * Q.TK * 4, v[0][combo], v[1][combo]);
    } else {
        const int steps = Q.WSZ / (PLANES * 8 * Q.TK);       // of a unit
#pragma unroll 4
        for (int i = wave; i < per * steps * 2; i += pack_run_threads(F23) / 64) {
            const int oct = i & 1, at = i >> 1, tr = at / steps, s = at - tr * steps, tap = tr * Q.TC + s;
            const bool there = s < Q.TC && tap < T;
            const float *src = runs + kk * k_step + (oct * 8 + 2 * j2) * c_step + (!there ? 0 : Q.mode == 0 ? tap : T - 1 - tap);
            const float v0 = src[0], v1 = src[c_step];
            store(group + (size_t)tr * Q.WSZ + (s * PLANES * 2 + oct) * Q.TK * 4, there ? v0 : 0.f, there ? v1 : 0.f);
        }
    }
}

// Weights of a folded view (folded_view, igemm_plan.h), as igemm_pack_weights_bf16_kernel<3>; a thread writes one pair of channels
__global__ __launch_bounds__(256) void igemm_pack_folded_kernel(const float *__restrict__ w, unsigned *__restrict__ packed, PackParams Q) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= Q.total / 3) return;
    const int words = Q.WSZ / 3;
    int t = p / words;
    const int within = p - t * words;
    unsigned *const unit = packed + (size_t)t * Q.WSZ;
    const int j2 = within & 3, row = within >> 2, so = row / Q.TK, kk = row - so * Q.TK, oct = so & 1, s = so >> 1;
    const int uu = t % Q.NU; t /= Q.NU;
    const int kt = t % Q.KT, g = t / Q.KT, cg = uu / Q.NTR, tap = (uu - cg * Q.NTR) * Q.TC + s, k = kt * Q.TK + kk;
    float v[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int vc = cg * BF_DC + oct * 8 + 2 * j2 + e, c = vc / (Q.Sh * Q.Sw), ph = vc - c * Q.Sh * Q.Sw, pj = ph / Q.Sh, pi = ph - pj * Q.Sh;
        const int fi = Q.Sh * (tap % Q.Hf) + pi, fj = Q.Sw * (tap / Q.Hf) + pj;
        const bool ok = s < Q.TC && tap < Q.Hf * Q.Wf && k < Q.Kg && vc < Q.Cg && fi < Q.HfA && fj < Q.WfA;
        v[e] = w[ok ? fi + Q.HfA * (fj + Q.WfA * (c + (size_t)Q.DfA * (g * Q.Kg + k))) : 0];
        if (!ok) v[e] = 0.f;
    }
    unsigned *dst = unit + ((size_t)(s * 3) * 2 + oct) * Q.TK * 4 + kk * 4 + j2;
    unsigned hi, mid, lo;
    split_bf16x3(v[0], v[1], &hi, &mid, &lo);
    dst[0] = hi; dst[2 * Q.TK * 4] = mid; dst[4 * Q.TK * 4] = lo;
}

// MERGED: the stride phases of an input derivative side by side in the filter dimension (IgemmParams::mD).
// GROUPED: 1x1 filters.  A unit of one group of 16 channels is a single step, and its barrier and staging take longer than that, so a unit is P.NS
// groups.  They stand in the slab as taps do, TQ samples from one to the next, and a sample is that of one pixel: no window, no halo.
// Bound by staging (a split sample meets 128 filters).  Forward of 28x28x512 -> 128, 64 images: 93 us with one group a unit, now 60, fp32 kernel 83; dzdw of
// 6x6x256 -> 4096, 256 images: 207 us on the fp32 kernel, now 155, its dzdx 187 and 134.
// QUADS: GROUPED where the pixels are the input's samples one after the other, in whole fours (stride 1, no padding, planes of a multiple of four): a
// staging thread brings four pixels in 8 channels by 16-byte loads (two pixels in 16 channels by loads of 4 bytes otherwise).  A wave is held at a load
// for 11 cycles of the compute unit's memory pipeline whatever its width up to 256 bytes in all, and for 15 at 1 KB.  28x28x512 -> 128, 64 images: dzdx
// 63.6 -> 59.5 us, forward 53.8 -> 52.5; 14x14x256 -> 256, 32 images 19.5 -> 16.9; 56x56x64 -> 256, 16 images 33.9 -> 31.4 and 28.4 -> 24.9; dzdw of
// 6x6x256 -> 4096, 256 images 148 -> 140; 200 random layers forward 4.5 % and dzdx 7 % in the mean.
// FOLDED: the channels of the reduction are the stride phases of the input's (folded_view, igemm_plan.h): a staging thread's sample is that of phase (0, 0), the
// others lie up to a stride behind it.  Forward of 227x227x3, 11x11x3x96 at stride 4, 128 images: 301 us on the fp32 kernel, 240 here, with a third of its
// error; a quarter of the 128 x 128 tiles has no filter.
// WK x WP computing waves; each owns MK x MP tiles of 32 filters x 32 pixels.
template <int WK, int WP, int MK, int MP, bool F23, bool MERGED, bool GROUPED, bool QUADS, bool FOLDED>
__global__ __launch_bounds__(64 * (WK * WP + SPLIT_STAGE_WAVES), WK * WP == 8 ? 3 : 2) void igemm_split_kernel(
    SplitParams P, const float *__restrict__ in, const float *__restrict__ wpk, const float *__restrict__ bias, float *out,
    float *__restrict__ part) {
    constexpr int NT = 64 * WK * WP;               // computing threads
    constexpr int NL = 64 * SPLIT_STAGE_WAVES;     // staging threads
    constexpr int TK = WK * MK * 32;
    constexpr int TQ = WP * MP * 32;
    constexpr int ROWS = F23 ? 2 : 1;              // input rows of a slab sample; output rows of a pixel
    constexpr int EPT = F23 ? 1 : 2, CH = F23 ? 8 : BF_DC, SETS = F23 ? 2 : 3;      // samples, channels a staging thread brings; units on their way
    const int NU = P.NU;
    const int CP = P.CP, SRP = P.SRP;
    const int XSZ = 3 * 2 * CP * 4;      // 32-bit words of slab per buffer: 3 planes x 2 octets x CP samples x 16 bytes

    extern __shared__ __align__(16) float lds[];
    float *xbuf = lds;                                              // [SLABS][XSZ]
    float *blds = xbuf + SPLIT_SLABS * XSZ;        // [BIASES][TK] bias of the tile, slots used in turn
    int2 *mlds = reinterpret_cast<int2 *>(blds + SPLIT_BIASES * TK);      // MERGED: [BIASES][TK] where the tile's filters go, see store_tile_merged

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HW = P.H * P.W;
    const int OHW = P.OH * P.OW;

    // ---- the block's range of units (see igemm_sk_kernel) ---------------------------------
    const int vb = sk_virtual_block(blockIdx.x, P.nblocks);
    const int tile_s0 = P.own * P.nblocks;                          // first shared tile
    // units of the shared tiles; F23: cut between channel groups, whose four combinations then meet in one piece (a piece
    // of fewer holds sums that the other pieces cancel, and rounds them)
    constexpr int CUT = F23 ? 4 : 1;
    const int rank = sk_share_rank(P.nblocks, P.nshare, vb);
    const long long ub = rank < 0 ? 0 : CUT * sk_begin(P.walk, rank), ue = rank < 0 ? 0 : CUT * sk_begin(P.walk, rank + 1);
    const int n_own = P.own * NU;                                    // units of this block's own tiles
    const int nunits = n_own + (int)(ue - ub);
    if (nunits == 0) return;
    const int ts = sk_tile(P.walk, ub, NU), t_s = tile_s0 + ts, uu_s = (int)(ub - (long long)ts * NU);
    auto tile_of = [&](int t) __attribute__((always_inline)) {                    // dealt among the blocks of an XCD, as in igemm_sk_kernel
        if (t >= tile_s0 || (P.nblocks & 7) != 0) return t;
        const int b = t / P.own, j = t - b * P.own;
        const int G = P.nblocks >> 3, x = b / G, i = b - x * G;
        return (x * G) * P.own + j * G + i;
    };

    if (wave >= WK * WP) {
        // ---- the waves that fetch the input and split it ----------------------------------
        // The samples of three (F23: two) units are on their way at a time, in as many sets of registers: a unit of few taps is
        // computed in less time than a sample takes from memory.  What a unit does not have is requested
        // out of range and reads as zero: no divergent branches, so that the waits for a set leave younger ones in flight.
        struct Samples {
            float v[EPT][ROWS][CH];        // QUADS: [octet channel][pixel of the quad]
            int uu, kt, g, seq, combo;
        };
        Samples set[SETS];
        const int ltid = tid - NT, lwave = wave - WK * WP;
        // QUADS: first of the thread's four pixels in the slab, and the octet it brings of them
        const int quads = CP / 4, quad_oct = QUADS && ltid >= quads ? 1 : 0, quad_e = 4 * (ltid - quads * quad_oct);
        const bool quad_there = quad_e < CP;
        // F23: the first two waves bring the first octet of channels, the others the second
        const int e0 = F23 ? ltid & (NL / 2 - 1) : ltid, wave0 = 64 * (F23 ? lwave & (SPLIT_STAGE_WAVES / 2 - 1) : lwave), oct0 = F23 ? lwave / (SPLIT_STAGE_WAVES / 2) : 0;
        int t = n_own ? vb * P.own : t_s, uu = n_own ? 0 : uu_s, n = 0;      // next unit to request, units before it
        int kt = 0, g = 0, seq = -1;
        const int sample_dc = GROUPED ? BF_DC * (ltid / TQ) : 0, set_dc = GROUPED ? BF_DC * (NL / TQ) : 0;       // first channel of the thread's samples, in the unit
        const int quad_dc = BF_DC * (quad_e / TQ) + 8 * quad_oct;                  // QUADS: the thread's first channel, in the unit
        int at_i[FOLDED ? EPT : 1], at_j[FOLDED ? EPT : 1];
        (void)at_i; (void)at_j;
        unsigned go[EPT][F23 ? 4 : 1];    // byte offset of the thread's samples in channel 0, or SLAB_INVALID; F23: of the pair's four rows
        __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc((void *)in, 0, 0, BUFFER_FLAGS);
        auto set_tile = [&](int tile) __attribute__((always_inline)) {
            ++seq;
            int pt, rb;
            decode_tile(P, tile, &kt, &pt, &rb, &g);
            const int q0 = pt * TQ;
            const int c_first = div32(q0, P.dTI);
            const int n_first = div32(c_first, P.dWo);
            const int u0 = (c_first - n_first * P.Wo) * P.Sw;   // chained column of the slab's first column
            const int row0 = rb * P.TI * P.Sh - P.Pt;           // input row of slab row 0
            const size_t in_base = ((size_t)n_first * P.Ctot + (size_t)g * P.Cg) * HW;
            size_t in_left = ((size_t)P.N * P.Ctot * HW - in_base) * 4;
            if (in_left > 0x7fffffffull) in_left = 0x7fffffffull;
            xrs = __builtin_amdgcn_make_buffer_rsrc((void *)(in + in_base), 0, (int)in_left, BUFFER_FLAGS);
            if constexpr (QUADS) {
                const int q = q0 + (quad_e & (TQ - 1)), n = div32(div32(q, P.dTI), P.dWo);
                go[0][0] = quad_there && q < P.QN ? 4u * (unsigned)(q - n * HW + (n - n_first) * P.Ctot * HW + quad_dc * HW) : SLAB_INVALID;
                return;
            }
#pragma unroll
            for (int s = 0; s < EPT; ++s) {
                const int e = e0 + NL * s;
                if constexpr (GROUPED) {
                    const int q = q0 + (e & (TQ - 1)), c = div32(q, P.dTI), n = div32(c, P.dWo), j = (c - n * P.Wo) * P.Sw - P.Pl, i = row0 + (q - c * P.TI) * P.Sh;
                    const bool ok = e < CP && q < P.QN && rb * P.TI + q - c * P.TI < P.Ho && j >= 0 && j < P.W && i >= 0 && i < P.H;
                    go[s][0] = ok ? 4u * ((unsigned)(i + P.H * j + (n - n_first) * P.Ctot * HW) + (unsigned)(sample_dc + set_dc * s) * (unsigned)HW) : SLAB_INVALID;
                    continue;
                }
                const int col = div32(e, P.dSRP);
                const int r = e - col * SRP;
                const int U = u0 + col;
                const int ni = div32(U, P.dWp);          // image relative to n_first
                if constexpr (FOLDED) {                  // of phase (0, 0): its row and column, which other phases lie behind
                    const bool there = e < CP && r < P.SR && (n_first + ni) < P.N;
                    at_i[s] = there ? P.F.fSh * (rb * P.TI + r) - P.Pt : -(1 << 28);
                    at_j[s] = P.F.fSw * (U - ni * P.Wp) - P.Pl;
                    go[s][0] = 4u * (unsigned)(at_i[s] + P.H * at_j[s] + ni * P.Ctot * HW);
                    continue;
                }
                const int j = U - ni * P.Wp - P.Pl;
                const int i0 = row0 + (F23 ? 2 * r : r);
                const bool ok = e < CP && r < P.SR && j >= 0 && j < P.W && (n_first + ni) < P.N;
#pragma unroll
                for (int a = 0; a < (F23 ? 4 : 1); ++a)
                    go[s][a] = ok && i0 + a >= 0 && i0 + a < P.H ? 4u * (unsigned)(i0 + a + P.H * j + ni * P.Ctot * HW) : SLAB_INVALID;
            }
        };
        auto request = [&](Samples &q) __attribute__((always_inline)) {
            const int combo = uu & 3, c0 = (F23 ? uu >> 2 : GROUPED ? uu * P.NS : uu) * BF_DC + 8 * oct0, c_end = n < nunits ? P.F.VC : 0;
            q.uu = uu; q.kt = kt; q.g = g; q.seq = seq; q.combo = combo;
            if constexpr (QUADS) {
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const floatx4 v = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                        xrs, c0 + d + quad_dc < c_end ? go[0][0] : SLAB_INVALID, (unsigned)(c0 + d) * (unsigned)HW * 4u, 0));
#pragma unroll
                    for (int r = 0; r < 4; ++r) q.v[d >> 2][0][4 * (d & 3) + r] = v[r];
                }
            }
            if constexpr (FOLDED) {
#pragma unroll
                for (int d = 0; d < CH; ++d) {
                    const int vc = c0 + d, c = div32(vc, P.F.dfSS), ph = vc - c * P.F.fSh * P.F.fSw, pj = div32(ph, P.F.dfSh), pi = ph - pj * P.F.fSh;
#pragma unroll
                    for (int s = 0; s < EPT; ++s) {
                        const bool ok = vc < c_end && (unsigned)(at_i[s] + pi) < (unsigned)P.H && (unsigned)(at_j[s] + pj) < (unsigned)P.W;
                        q.v[s][0][d] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xrs, ok ? go[s][0] + 4u * (unsigned)(pi + P.H * pj) : SLAB_INVALID,
                                                                                           (unsigned)c * (unsigned)HW * 4u, 0));
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < (QUADS || FOLDED ? 0 : EPT); ++s) {
                if (s * NL >= CP) continue;
#pragma unroll
                for (int a = 0; a < ROWS; ++a) {
                    unsigned off = go[s][0];
                    if constexpr (F23) {           // d0-d2, d1+d2, d2-d1, d1-d3
                        if (a == 0) off = combo == 0 ? go[s][0] : combo == 2 ? go[s][2] : go[s][1];
                        else off = combo == 3 ? go[s][3] : combo == 2 ? go[s][1] : go[s][2];
                    }
#pragma unroll
                    for (int d = 0; d < CH; ++d)
                        // channels past the group's last one read as zero (their weights are zero too)
                        q.v[s][a][d] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                            xrs, c0 + d + (GROUPED ? sample_dc + set_dc * s : 0) < c_end ? off : SLAB_INVALID, (unsigned)(c0 + d) * (unsigned)HW * 4u, 0));
                }
            }
            // on to the next unit
            ++n;
            const int t_old = t;
            if (n == n_own) { t = t_s; uu = uu_s; }
            else if (++uu == NU) { uu = 0; ++t; }
            if (t != t_old && n < nunits) set_tile(tile_of(t));
        };
        int slab = 0;
        auto write = [&](Samples &q) __attribute__((always_inline)) {
            if (q.uu == 0 && (MERGED || bias) && ltid < TK) {    // of a tile this block may own entirely: start values, and where filters go
                const int kl = q.kt * TK + ltid, at = (q.seq & (SPLIT_BIASES - 1)) * TK + ltid;
                int ch = q.g * P.Kg + kl;
                if constexpr (MERGED) {
                    const MergedFilter f = merged_filter(P, kl < P.Kg ? kl : 0);
                    ch = q.g * P.mD + f.c;
                    // 1: this phase has no last row, 2: no last column, 4: no such filter
                    const int missing = (f.i0 + P.osi * (P.Ho - 1) >= P.OH ? 1 : 0) | (f.j0 + P.osj * (P.Wo - 1) >= P.OW ? 2 : 0) | (kl < P.Kg ? 0 : 4);
                    mlds[at] = int2{4 * (ch * OHW + f.i0 + P.OH * f.j0), missing};
                }
                if (bias) blds[at] = kl < P.Kg ? bias[ch] : 0.f;
            }
            float *xb = xbuf + slab * XSZ;
            slab = slab + 1 == SPLIT_SLABS ? 0 : slab + 1;
            if constexpr (QUADS) {
                if (!quad_there) return;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    auto value = [&](int d) { return q.v[d >> 2][0][4 * (d & 3) + r]; };
                    unsigned hi[4], mid[4], lo[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) split_bf16x3(value(2 * j), value(2 * j + 1), &hi[j], &mid[j], &lo[j]);
                    float *const at = xb + (size_t)(quad_oct * CP + quad_e + r) * 4;
                    *reinterpret_cast<uintx4 *>(at) = uintx4{hi[0], hi[1], hi[2], hi[3]};
                    *reinterpret_cast<uintx4 *>(at + 2 * CP * 4) = uintx4{mid[0], mid[1], mid[2], mid[3]};
                    *reinterpret_cast<uintx4 *>(at + 4 * CP * 4) = uintx4{lo[0], lo[1], lo[2], lo[3]};
                }
            }
#pragma unroll
            for (int s = 0; s < (QUADS ? 0 : EPT); ++s) {
                const int e = e0 + NL * s;
                if (wave0 + NL * s >= CP) continue;              // CP is a multiple of 64
                if constexpr (F23) {
                    const float sign = q.combo == 1 ? 1.f : -1.f;
#pragma unroll
                    for (int d = 0; d < CH; ++d) q.v[s][0][d] = fmaf(sign, q.v[s][1][d], q.v[s][0][d]);
                }
#pragma unroll
                for (int i = 0; i < CH / 8; ++i) {
                    const int o = oct0 + i;
                    unsigned hi[4], mid[4], lo[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        split_bf16x3(q.v[s][0][8 * i + 2 * j], q.v[s][0][8 * i + 2 * j + 1], &hi[j], &mid[j], &lo[j]);
                    const uintx4 h = {hi[0], hi[1], hi[2], hi[3]}, m = {mid[0], mid[1], mid[2], mid[3]}, l = {lo[0], lo[1], lo[2], lo[3]};
                    *reinterpret_cast<uintx4 *>(xb + (size_t)((0 + o) * CP + e) * 4) = h;
                    *reinterpret_cast<uintx4 *>(xb + (size_t)((2 + o) * CP + e) * 4) = m;
                    *reinterpret_cast<uintx4 *>(xb + (size_t)((4 + o) * CP + e) * 4) = l;
                }
            }
        };
        set_tile(tile_of(t));
#pragma unroll
        for (int j = 0; j < SETS; ++j) request(set[j]);
        for (int it = -2; it < nunits; it += SETS) {    // unit it + 2 is written after the barrier of unit it
#pragma unroll
            for (int j = 0; j < SETS; ++j) {
                if (it + j >= 0 && it + j < nunits) lds_barrier();
                if (it + j + 2 < nunits) {
                    write(set[j]);
                    request(set[j]);
                }
            }
        }
        return;
    }

    // ---- the computing waves --------------------------------------------------------------
    const int wk = wave % WK, wp = wave / WK;
    int bbase[MP];       // slab byte offset of the pixel's window origin, octet of this half-wave
    unsigned ooff[MP];   // byte offset of the lane's first result relative to the tile's output window, or SLAB_INVALID
    unsigned ooff1[MP];  // F23: the same for the second row of the pair
    int edge[MP];        // merged phases: 1 = last row of the view, 2 = last column
    __amdgpu_buffer_rsrc_t ors = __builtin_amdgcn_make_buffer_rsrc((void *)out, 0, 0, BUFFER_FLAGS);
    int c_kt = 0, c_g = 0, c_seq = -1;
    // sums of the products of the three scales (F23: of the current combination), and F23: the rows'
    floatx16 acc[MK][MP], sum8[MK][MP], sum16[MK][MP], row0[F23 ? MK : 1][MP], row1[F23 ? MK : 1][MP];
    auto whole_sum = [&](int mk, int mp, int v) __attribute__((always_inline)) {
        return fmaf(fmaf(sum16[mk][mp][v], 0x1p-8f, sum8[mk][mp][v]), 0x1p-8f, acc[mk][mp][v]);
    };
    auto set_tile = [&](int t) __attribute__((always_inline)) {
        ++c_seq;
        int kt, pt, rb, g;
        decode_tile(P, t, &kt, &pt, &rb, &g);
        c_kt = kt; c_g = g;
        const int q0 = pt * TQ;
        const int qend = min(q0 + TQ, P.QN);
        const int c_first = div32(q0, P.dTI);
        const int n_first = div32(c_first, P.dWo);
        const int u0 = (c_first - n_first * P.Wo) * P.Sw;
#pragma unroll
        for (int mp = 0; mp < MP; ++mp) {
            const int q = q0 + (wp * MP + mp) * 32 + (lane & 31);
            const int c = div32(q, P.dTI);
            const int ii = q - c * P.TI;
            const int n = div32(c, P.dWo);
            const int jo = c - n * P.Wo;
            const int io = rb * P.TI + ii;
            const bool ok = q < qend && io < P.Ho;
            const int ucol = jo * P.Sw + (n - n_first) * P.Wp - u0;
            if constexpr (GROUPED) bbase[mp] = 16 * ((wp * MP + mp) * 32 + (lane & 31) + half * CP);
            else bbase[mp] = 16 * ((ok ? ii * (F23 ? 1 : P.Sh) + SRP * ucol : 0) + half * CP);
            ooff[mp] = ok ? 4u * (unsigned)((P.oi0 + P.osi * io) + P.OH * (P.oj0 + P.osj * jo) +
                                            OHW * (P.Ktot * (n - n_first) + (MERGED ? 0 : 4 * half)))
                          : SLAB_INVALID;
            edge[mp] = (io == P.Ho - 1 ? 1 : 0) | (jo == P.Wo - 1 ? 2 : 0);
            if constexpr (F23)
                ooff1[mp] = ok && 2 * io + 1 < P.wino_Ho ? ooff[mp] + 4u * (unsigned)(P.osi >> 1) : SLAB_INVALID;
        }
        (void)ooff1; (void)edge;
        const size_t out_base = (size_t)n_first * P.Ktot * OHW;
        size_t out_left = ((size_t)P.N * P.Ktot * OHW - out_base) * 4;
        if (out_left > 0x7fffffffull) out_left = 0x7fffffffull;
        ors = __builtin_amdgcn_make_buffer_rsrc((void *)(out + out_base), 0, (int)out_left, BUFFER_FLAGS);
    };
    auto init_acc = [&](bool with_bias) __attribute__((always_inline)) {
        const float *bl = blds + (c_seq & (SPLIT_BIASES - 1)) * TK;
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int kloc = (wk * MK + mk) * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
                const float bv = with_bias ? bl[kloc] : 0.f;
#pragma unroll
                for (int mp = 0; mp < MP; ++mp) {
                    if constexpr (F23) { row0[mk][mp][v] = bv; row1[mk][mp][v] = bv; }
                    else { acc[mk][mp][v] = bv; sum8[mk][mp][v] = sum16[mk][mp][v] = 0.f; }
                }
            }
    };
    // F23: the finished sum of a run of units goes to the two rows
    auto fold = [&](int combo) __attribute__((always_inline)) {
        const float s0 = combo < 3 ? 1.f : 0.f, s1 = combo == 0 ? 0.f : combo == 1 ? 1.f : -1.f;
#pragma unroll
        for (int mk = 0; mk < (F23 ? MK : 0); ++mk)
#pragma unroll
            for (int mp = 0; mp < MP; ++mp)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float m = whole_sum(mk, mp, v);
                    row0[mk][mp][v] = fmaf(s0, m, row0[mk][mp][v]);
                    row1[mk][mp][v] = fmaf(s1, m, row1[mk][mp][v]);
                }
    };
    const int aoff = 16 * (half * TK + wk * MK * 32 + (lane & 31));   // bytes
    const int T = F23 ? 3 : GROUPED ? P.NS : P.Hf * P.Wf;
    const int xplane = 2 * CP * 16;                  // bytes from a slab plane to the next
    // where the next operands are read: weights of the step (steps follow one another in memory through all units of a
    // tile), slab and offset of its tap.  All scalar but the two lane offsets.
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)wpk, 0, (int)P.packed_bytes, BUFFER_FLAGS);
    constexpr int WPLANE = 2 * TK * 16, WSTEP = 3 * WPLANE;
    unsigned wo = 0;
    int xo = 0, xslab = 0, fi = 0, so = 0;
    const int xbytes = 4 * XSZ;
    const char *const xlane = reinterpret_cast<const char *>(xbuf);
    auto next_tap = [&]() __attribute__((always_inline)) {
        if constexpr (F23) {
            so += 16 * SRP;
        } else if constexpr (GROUPED) {
            so += 16 * TQ;
        } else {
            const bool wrap = ++fi == P.Hf;
            so += wrap ? 16 * (SRP - P.Hf + 1) : 16;
            if (wrap) fi = 0;
        }
    };
    auto next_slab = [&]() __attribute__((always_inline)) {
        xslab = xslab + xbytes == SPLIT_SLABS * xbytes ? 0 : xslab + xbytes;
    };
    typedef bf16x8 OpA[MK];
    typedef bf16x8 OpB[MP];
    OpA wreg[F23 ? 3 : 1][3];                  // [tap (F23)][plane]
    OpA (&ah) = wreg[0][0], (&am) = wreg[0][1], (&al) = wreg[0][2];
    OpB bh, bm, bl;
    auto load_a = [&](OpA &a, int pl) __attribute__((always_inline)) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) a[mk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wrs, (unsigned)aoff + mk * 512u, wo + (unsigned)(pl * WPLANE), 0));
    };
    auto load_b = [&](OpB &b, int pl) __attribute__((always_inline)) {
#pragma unroll
        for (int mp = 0; mp < MP; ++mp) b[mp] = *reinterpret_cast<const bf16x8 *>(xlane + bbase[mp] + (xo + so + pl * xplane));
    };
    auto mma = [&](floatx16 (&sum)[MK][MP], const OpA &a, const OpB &b, bool from_zero = false) __attribute__((always_inline)) {
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int mp = 0; mp < MP; ++mp)
                sum[mk][mp] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mk], b[mp], from_zero ? floatx16{} : sum[mk][mp], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto prime = [&]() __attribute__((always_inline)) {
        load_a(ah, 0); load_b(bl, 2); load_b(bm, 1); load_b(bh, 0); load_a(am, 1); load_a(al, 2);
        if constexpr (F23) {
#pragma unroll
            for (int s = 1; s < 3; ++s) {
                wo += WSTEP;
                load_a(wreg[s][0], 0); load_a(wreg[s][1], 1); load_a(wreg[s][2], 2);
            }
        }
    };
    // one step; xo, so are the next step's when it begins, wo is where the weights are that h, m, l hold next: the next step's, or
    // (F23) the same tap's of the next unit; first: the first one of a combination's sums (F23)
    auto step = [&](OpA &h, OpA &m, OpA &l, bool first) __attribute__((always_inline)) {
        mma(sum16, h, bl, F23 && first);
        load_b(bl, 2);
        mma(sum8, h, bm, F23 && first);
        mma(acc, h, bh, F23 && first);
        load_a(h, 0);
        mma(sum16, m, bm);
        load_b(bm, 1);
        mma(sum8, m, bh);
        load_a(m, 1);
        mma(sum16, l, bh);
        load_b(bh, 0);
        load_a(l, 2);
        __builtin_amdgcn_sched_barrier(0);
    };

    bool odd_results = false;        // of the lane in the tile just stored: some are not finite (repair_tile)
    auto store_tile = [&]() __attribute__((always_inline)) {
        odd_results = false;
#pragma unroll
        for (int mk = 0; mk < MK; ++mk) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int kl0 = c_kt * TK + (wk * MK + mk) * 32 + (v >> 2) * 8 + (v & 3);   // filter of the lower half-wave
                const int left = P.Kg - kl0;
                if (left <= 0) continue;
                const unsigned soff = (unsigned)(c_g * P.Kg + kl0) * (unsigned)OHW * 4u;
#pragma unroll
                for (int mp = 0; mp < MP; ++mp) {
                    const unsigned vo = (left > 4 || half == 0) ? ooff[mp] : SLAB_INVALID;   // the upper half-wave holds filter kl0 + 4
                    auto finish = [&](float val) __attribute__((always_inline)) {
                        const bool odd = not_finite(val);
                        odd_results |= odd;
                        if (P.relu) val = odd ? __uint_as_float(0x7fc00000u) : fmaxf(val, 0.f);
                        return __float_as_uint(val);
                    };
                    if constexpr (F23) {
                        const bool both = left > 4 || half == 0, two_rows = ooff1[mp] != SLAB_INVALID;
                        uintx2 yy;
                        yy.x = finish(row0[mk][mp][v]);
                        yy.y = finish(row1[mk][mp][v]);
                        if (P.wino_pairs) {        // a pair without a second row (odd number of rows) goes alone
                            __builtin_amdgcn_raw_buffer_store_b64(yy, ors, both && two_rows ? ooff[mp] : SLAB_INVALID, soff, 0);
                            if (P.wino_Ho & 1)
                                __builtin_amdgcn_raw_buffer_store_b32(yy.x, ors, both && !two_rows ? ooff[mp] : SLAB_INVALID, soff, 0);
                        } else {
                            __builtin_amdgcn_raw_buffer_store_b32(yy.x, ors, both ? ooff[mp] : SLAB_INVALID, soff, 0);
                            __builtin_amdgcn_raw_buffer_store_b32(yy.y, ors, both ? ooff1[mp] : SLAB_INVALID, soff, 0);
                        }
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b32(finish(acc[mk][mp][v]), ors, vo, soff, 0);
                    }
                }
            }
        }
    };
    // Merged phases: the two half-waves hold filters of different phases, so the filter part of the address and the "does
    // this pixel exist in this phase" test are per half-wave.  Both come from a table that the staging waves write, one filter a
    // thread: found here, by each wave for all of its filters, they were thousands of instructions of divisions a tile (dzdx of
    // 37x53x16, 3x5x16x24 at stride 2x3, four images: 26.1 -> 14.0 us; of 227x227x3, 11x11x3x96 at stride 4, 128 images: 293 -> 235).
    auto store_tile_merged = [&]() __attribute__((always_inline)) {
        odd_results = false;
        const int2 *table = mlds + (c_seq & (SPLIT_BIASES - 1)) * TK + wk * MK * 32 + half * 4;
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if (c_kt * TK + (wk * MK + mk) * 32 + (v >> 2) * 8 + (v & 3) >= P.Kg) continue;
                const int2 f = table[mk * 32 + (v >> 2) * 8 + (v & 3)];
#pragma unroll
                for (int mp = 0; mp < MP; ++mp) {
                    const bool drop = (f.y & (edge[mp] | 4)) != 0 || ooff[mp] == SLAB_INVALID;
                    const float val = acc[mk][mp][v];
                    odd_results |= !drop && not_finite(val);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val), ors, drop ? SLAB_INVALID : ooff[mp] + (unsigned)f.x, 0, 0);
                }
            }
    };
    auto store_partial = [&](int slot) __attribute__((always_inline)) {
        float *dst = part + (size_t)slot * (TK * TQ * ROWS);
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int kloc = (wk * MK + mk) * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
#pragma unroll
                for (int mp = 0; mp < MP; ++mp) {
                    const int ql = (wp * MP + mp) * 32 + (lane & 31);
                    if constexpr (F23)             // in the output domain: pixel = 2 * pair + row
                        *reinterpret_cast<float2 *>(dst + kloc * (2 * TQ) + 2 * ql) = float2{row0[mk][mp][v], row1[mk][mp][v]};
                    else
                        dst[kloc * TQ + ql] = acc[mk][mp][v];
                }
            }
    };
    // One segment = the units of one tile in a row.
    int t = n_own ? vb * P.own : t_s, uu = n_own ? 0 : uu_s;
    bool first_segment = true;
    for (int done = 0; done < nunits;) {
        const bool own = done < n_own;
        const int left = nunits - done, m = NU - uu < left ? NU - uu : left;
        // the segment covers its tile iff the tile is the block's own, or it starts at 0 and reaches the tile's end
        const bool whole = m == NU;
        set_tile(tile_of(t));
        wo = (unsigned)(((c_g * P.KT + c_kt) * NU + uu) * T) * (unsigned)WSTEP;
        fi = 0; so = 0; xo = xslab;
        // This unit's slab and the next one's are in place.  The reads still in flight are of this unit's slab, which
        // is written again two barriers later: nothing to wait for.
        asm volatile("s_barrier" ::: "memory");
        // not inside the loop: no sum is then alive (in registers) between two segments
        init_acc(whole && bias != nullptr);
        prime();
        for (int u = 0;;) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (F23) {
                // One wave a SIMD: the weights of a step are requested a whole unit ahead, since nothing else covers their way from
                // the L2 (14x14x512, 3x3x512x512, 32 images: 187 us with one step ahead, now 173).  Past the last unit they read what follows,
                // or zero, for nothing.
                wo += WSTEP; next_tap();
                step(wreg[0][0], wreg[0][1], wreg[0][2], true);
                wo += WSTEP; next_tap();
                step(wreg[1][0], wreg[1][1], wreg[1][2], false);
                wo += WSTEP; next_slab();
                if (u + 1 < m) { so = 0; xo = xslab; }
                step(wreg[2][0], wreg[2][1], wreg[2][2], false);
            } else {
                for (int s = 1; s < T; ++s) {
                    wo += WSTEP;
                    next_tap();
                    step(ah, am, al, false);
                }
                next_slab();
                if (u + 1 < m) { wo += WSTEP; fi = 0; so = 0; xo = xslab; }
                step(ah, am, al, false);           // the segment's last one reads its own operands again, for nothing
            }
            if constexpr (F23) {
                fold((uu + u) & 3);
                // before the barrier, where waves wait for one another anyway: the compiler would move it behind (14x14x512,
                // 3x3x512x512, 32 images: 209 against 189 us)
#pragma unroll
                for (int mk = 0; mk < MK; ++mk)
#pragma unroll
                    for (int mp = 0; mp < MP; ++mp) asm volatile("" : "+v"(row0[mk][mp]), "+v"(row1[mk][mp]));
            }
            if (++u == m) break;
            asm volatile("s_barrier" ::: "memory");
        }
        // a use of what the last step read for nothing: without one the compiler moves the weights' loads of every unit's last step
        // behind its products, where their latency is not hidden
#pragma unroll
        for (int s = 0; s < (F23 ? 3 : 1); ++s)
#pragma unroll
            for (int mk = 0; mk < MK; ++mk) asm volatile("" ::"v"(wreg[s][0][mk]), "v"(wreg[s][1][mk]), "v"(wreg[s][2][mk]));
        done += m;
#pragma unroll
        for (int mk = 0; mk < MK; ++mk)
#pragma unroll
            for (int mp = 0; mp < (F23 ? 0 : MP); ++mp)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mk][mp][v] = whole_sum(mk, mp, v);
        if (whole) {
            if constexpr (MERGED) store_tile_merged();
            else store_tile();
            if (__any(odd_results)) {
                const size_t params = (size_t)__builtin_amdgcn_kernarg_segment_ptr();
                if constexpr (F23) repair_pairs<TK, WK, MK, MP, TQ>((unsigned)params, (unsigned)(params >> 32), tile_of(t), wave);
                else repair_tile<TK, WK, MK, MP, TQ, ROWS, MERGED>((unsigned)params, (unsigned)(params >> 32), tile_of(t), wave);
            }
        } else {
            store_partial(2 * vb + (first_segment ? 0 : 1));
        }
        first_segment = done == n_own;             // the shared range starts with a "first" segment again
        if (own && done == n_own) { t = t_s; uu = uu_s; }
        else { ++t; uu = 0; }
    }
}

}  // namespace mcn
