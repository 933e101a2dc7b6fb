// Host-side planning for the implicit-GEMM kernel: which instantiation, how the
// pixels are cut into row blocks and tiles, how the reduction is cut into units,
// how large the LDS buffers are, and how many resident blocks share the work.
#pragma once
#include <stdint.h>
#include <stddef.h>
#include <stdlib.h>
#include <math.h>
#include <algorithm>
#include "geom.h"
#include "kern_direct.h"
#include "kern_igemm.h"
#include "kern_igemm_bf16.h"
#include "kern_igemm_split.h"
#include "kern_small.h"

namespace mcn {

// One convolution "view": the sum the kernel evaluates (see kern_igemm.h).
struct ConvView {
    int H, W, N, Ctot, Cg;          // input array of the view
    int Ho, Wo, Ktot, Kg, G;        // output pixels computed, output channels
    int Hf, Wf, Sh, Sw, Pt, Pl;
    int OH, OW, oi0, osi, oj0, osj; // placement of the view's output pixels in the output array
    // weight packing (PackParams): mode, shape of the caller's filter array, stride phase
    int pack_mode, HfA, WfA, DfA, pSh, pSw, pi, pj, ldk;
    // all stride phases of an input derivative merged into one view (pack mode 3; kern_igemm.h)
    int mD, mPt, mPl, B0i, B0j;
    // strided view with the input's stride phases as channels (folded_view): the strides; 0 otherwise
    int fSh, fSw;
};

inline ConvView forward_view(const Geom &g) {
    ConvView v = {};
    v.H = g.H; v.W = g.W; v.N = g.N; v.Ctot = g.D; v.Cg = g.Df;
    v.Ho = g.Ho; v.Wo = g.Wo; v.Ktot = g.K; v.Kg = g.Kg; v.G = g.G;
    v.Hf = g.Hf; v.Wf = g.Wf; v.Sh = g.Sh; v.Sw = g.Sw; v.Pt = g.Pt; v.Pl = g.Pl;
    v.OH = g.Ho; v.OW = g.Wo; v.oi0 = 0; v.osi = 1; v.oj0 = 0; v.osj = 1;
    v.pack_mode = 0; v.HfA = g.Hf; v.WfA = g.Wf; v.DfA = g.Df;
    return v;
}

// Input derivative, one stride phase (pi, pj), 0 <= pi < Sh, 0 <= pj < Sw  (Sec. 6.1 dz/dX, in the
// gather form of Sec. 6.2):  dzdx[i,j] = sum_{fi,fj,k} w[fi,fj,.,k] dzdy[(i+Pt-fi)/Sh, (j+Pl-fj)/Sw, k]
// over the taps for which the divisions are exact.  Rows i = i0 + Sh*m with i0 = (pi-Pt) mod Sh
// only see taps fi = pi + Sh*a; with t = A-1-a this is a stride-1 sum over dzdy with A taps and top
// pad A-1-b0, b0 = (i0+Pt-pi)/Sh.  Returns false if the phase has no taps or no rows (nothing to do:
// those samples of dzdx are zero).
inline bool backward_data_view(const Geom &g, int pi, int pj, ConvView *out) {
    const int A = pi < g.Hf ? (g.Hf - pi + g.Sh - 1) / g.Sh : 0;
    const int Bt = pj < g.Wf ? (g.Wf - pj + g.Sw - 1) / g.Sw : 0;
    const int i0 = ((pi - g.Pt) % g.Sh + g.Sh) % g.Sh;
    const int j0 = ((pj - g.Pl) % g.Sw + g.Sw) % g.Sw;
    const int Mi = i0 < g.H ? (g.H - i0 + g.Sh - 1) / g.Sh : 0;
    const int Mj = j0 < g.W ? (g.W - j0 + g.Sw - 1) / g.Sw : 0;
    if (A == 0 || Bt == 0 || Mi == 0 || Mj == 0) return false;
    const int b0 = (i0 + g.Pt - pi) / g.Sh, d0 = (j0 + g.Pl - pj) / g.Sw;   // exact divisions
    ConvView v = {};
    v.H = g.Ho; v.W = g.Wo; v.N = g.N; v.Ctot = g.K; v.Cg = g.Kg;
    v.Ho = Mi; v.Wo = Mj; v.Ktot = g.D; v.Kg = g.Df; v.G = g.G;
    v.Hf = A; v.Wf = Bt; v.Sh = 1; v.Sw = 1; v.Pt = A - 1 - b0; v.Pl = Bt - 1 - d0;
    v.OH = g.H; v.OW = g.W; v.oi0 = i0; v.osi = g.Sh; v.oj0 = j0; v.osj = g.Sw;
    v.pack_mode = 1; v.HfA = g.Hf; v.WfA = g.Wf; v.DfA = g.Df; v.pSh = g.Sh; v.pSw = g.Sw; v.pi = pi; v.pj = pj;
    *out = v;
    return true;
}

// Input derivative with all Sh*Sw stride phases in ONE view: the phases read the same dzdy, so they can
// share the slab and sit side by side in the "filter" dimension of the GEMM (merged filter = channel
// + D' * phase).  Worth it when a phase alone would leave most of a 32-row MFMA tile empty (few
// channels per group, e.g. the derivative with respect to an image with 3 channels).  Per direction
// the phases' tap ranges are put into one window: output row i0 + Sh*m of phase pi meets dzdy rows
// m + b0 - a, a = 0..A-1; with B0 = max b0 the window covers rows m + B0 - t, t = 0..TH-1.  Phases
// without taps (stride larger than the filter) are all-zero filters, so nothing is left to fill.
inline bool merged_backward_data_view(const Geom &g, ConvView *out) {
    if (g.Sh * g.Sw < 2 || g.Df > 16 || g.Df * g.Sh * g.Sw > 1024) return false;
    int B0[2] = {0, 0}, TH[2] = {1, 1};
    const int Hf[2] = {g.Hf, g.Wf}, S[2] = {g.Sh, g.Sw}, Pd[2] = {g.Pt, g.Pl};
    for (int d = 0; d < 2; ++d) {
        bool any = false;
        for (int pi = 0; pi < S[d]; ++pi) {
            if (pi >= Hf[d]) continue;
            const int i0 = ((pi - Pd[d]) % S[d] + S[d]) % S[d];
            const int b0 = (i0 + Pd[d] - pi) / S[d];
            if (!any || b0 > B0[d]) B0[d] = b0;
            any = true;
        }
        for (int pi = 0; pi < S[d]; ++pi) {
            if (pi >= Hf[d]) continue;
            const int A = (Hf[d] - pi + S[d] - 1) / S[d];
            const int i0 = ((pi - Pd[d]) % S[d] + S[d]) % S[d];
            const int b0 = (i0 + Pd[d] - pi) / S[d];
            if (A + B0[d] - b0 > TH[d]) TH[d] = A + B0[d] - b0;
        }
    }
    ConvView v = {};
    v.H = g.Ho; v.W = g.Wo; v.N = g.N; v.Ctot = g.K; v.Cg = g.Kg;
    v.Ho = (g.H + g.Sh - 1) / g.Sh; v.Wo = (g.W + g.Sw - 1) / g.Sw;
    v.Ktot = g.D; v.Kg = g.Df * g.Sh * g.Sw; v.G = g.G;
    v.Hf = TH[0]; v.Wf = TH[1]; v.Sh = 1; v.Sw = 1; v.Pt = TH[0] - 1 - B0[0]; v.Pl = TH[1] - 1 - B0[1];
    v.OH = g.H; v.OW = g.W; v.oi0 = 0; v.osi = g.Sh; v.oj0 = 0; v.osj = g.Sw;
    v.pack_mode = 3; v.HfA = g.Hf; v.WfA = g.Wf; v.DfA = g.Df; v.pSh = g.Sh; v.pSw = g.Sw;
    v.mD = g.Df; v.mPt = g.Pt; v.mPl = g.Pl; v.B0i = B0[0]; v.B0j = B0[1];
    *out = v;
    return true;
}

// A strided forward view of few channels with the stride phases of its input as channels of their own (pack mode 4): channel c of the view's stride-1 sum is
// row phase pi and column phase pj of input channel c / (Sh*Sw), c % (Sh*Sw) = pi + Sh*pj, its sample (i, j) is the input's (Sh*i + pi - Pt, Sw*j + pj - Pl), and its
// tap (a, b) the filter's (Sh*a + pi, Sw*b + pj), zero past the filter's edge.  Three channels fill 3 of the 16 that an MFMA on bf16 takes; so folded, 11x11x3 at stride 4
// is 48 channels of 3x3 taps, 84 % of them real.
inline bool folded_view(const ConvView &v, ConvView *out) {
    if (v.pack_mode != 0 || v.mD || v.Cg >= 16 || v.Sh * v.Sw < 2 || v.Sh > 8 || v.Sw > 8 || v.Pt < 0 || v.Pl < 0) return false;
    ConvView f = v;
    f.Hf = (v.Hf + v.Sh - 1) / v.Sh; f.Wf = (v.Wf + v.Sw - 1) / v.Sw; f.Sh = f.Sw = 1; f.Cg = v.Cg * v.Sh * v.Sw;
    f.fSh = v.Sh; f.fSw = v.Sw; f.pack_mode = 4;
    // Nine taps or more, three of ten products with zeros at most, 128 pixels for every compute unit.  Forward of 227x227x3, 11x11x3x96 at stride 4, 128 images 301 -> 240 us
    // on 128 x 128 tiles (96 filters: a quarter of them empty), 9x9 at stride 3 100 -> 83; with fewer taps a tile's reduction is shorter than its way in and out (6x6 at
    // stride 3, 32 channels of four taps, 61 -> 76 us), with more zeros they cost what bf16 saves (7x7x3 at stride 2 85 -> 94, 5x5 63 -> 78).
    const int64_t taps = (int64_t)f.Hf * f.Wf;
    if (taps < 9 || 7 * ((f.Cg + 15) / 16 * 16 * taps) > 10 * (int64_t)v.Cg * v.Hf * v.Wf || (int64_t)v.Ho * v.Wo * v.N < 32768) return false;
    *out = f;
    return true;
}

// Fully-connected case (Sec. 4.1: a filter as large as the input, one output sample per image,
// no padding, one group).  With R = H*W*D the three passes are plain matrix products of
// X (R x N), F (R x K) and dY (K x N), all stored with their first index fastest:
//   Y = F^T X + b,   dX = F dY,   dF = X dY^T.
inline bool is_fully_connected(const Geom &g) {
    return g.G == 1 && g.H == g.Hf && g.W == g.Wf && g.Pt == 0 && g.Pb == 0 && g.Pl == 0 && g.Pr == 0;
}
inline ConvView fc_view_1x1(int64_t R, int C, int K) {
    ConvView v = {};
    v.H = (int)R; v.W = 1; v.N = 1; v.Ctot = C; v.Cg = C;
    v.Ho = (int)R; v.Wo = 1; v.Ktot = K; v.Kg = K; v.G = 1;
    v.Hf = 1; v.Wf = 1; v.Sh = 1; v.Sw = 1; v.Pt = 0; v.Pl = 0;
    v.OH = (int)R; v.OW = 1; v.oi0 = 0; v.osi = 1; v.oj0 = 0; v.osj = 1;
    v.pack_mode = 0; v.HfA = 1; v.WfA = 1; v.DfA = C;
    return v;
}
// Y[k][n] = sum_r F[r][k] X[r][n]: the split-K kernel with the coefficients r as "pixels", the
// images as "filters" and the filters as "channels" (both operands contiguous along r).
inline ConvView fc_forward_view(const Geom &g) { return fc_view_1x1((int64_t)g.H * g.W * g.D, g.K, g.N); }
// dX[r][n] = sum_k F[r][k] dY[k][n]: a 1x1 convolution over the "image" F with R pixels and K
// channels, whose N filters are the columns of dY.
inline ConvView fc_backward_data_view(const Geom &g) { return fc_view_1x1((int64_t)g.H * g.W * g.D, g.K, g.N); }
// dF[r][k] = sum_n X[r][n] dY[k][n]: a 1x1 convolution over the "image" X with R pixels and N
// channels, whose K filters are the rows of dY (read transposed by the packing pass).
inline ConvView fc_backward_filter_view(const Geom &g) {
    ConvView v = fc_view_1x1((int64_t)g.H * g.W * g.D, g.N, g.K);
    v.pack_mode = 2; v.ldk = g.K;
    return v;
}

// IG_W*: the WINO kernels (filters x pairs of output rows)
// IG_96x256: eight waves of 96 filters x 32 pixels each, for 65 to 96 filters per group (a quarter fewer MFMAs than 128-filter tiles)
enum IgemmShape { IG_128x256 = 0, IG_64x512 = 1, IG_32x256 = 2, IG_64x256 = 3, IG_W128x128 = 4, IG_W64x256 = 5, IG_96x256 = 6,
                  IG_S64x256 = 7, IG_S128x128 = 8, IG_S128x64 = 9,     // three-plane kernel only
                  IG_NONE = -1 };

struct IgemmPlan {
    int shape;          // IgemmShape
    bool bf16;          // operands rounded to bf16 (kern_igemm_bf16.h); sizes below are then in 32-bit words
    int planes;         // bf16: 1; 2 = operands split into hi and lo bf16 planes, three products each; 3 = fp32 operands in three planes
    int fixed;          // index into IGEMM_FIXED: an instantiation with compile-time filter size (0 = none)
    int TK, TQ, NT;
    IgemmParams P;
    PackParams Q;
    PlainView V;        // three planes
    FoldedChannels F;   // three planes
    size_t lds_bytes;
    size_t packed_floats;
    size_t partial_floats;   // 2 slots of TK*TQ per resident block
    double score;            // the planner's cost figure of the chosen row-block height (lower is better)
};

constexpr size_t IGEMM_LDS_LIMIT = 160 * 1024;
constexpr int IGEMM_LOADER_WAVES = 4;     // fetching waves per block
// Instantiations with a compile-time filter size and channel count per unit: every LDS offset of
// the MFMA loop is then an immediate or one of a few hoisted sums, against an offset-table read and
// several address instructions per step in the general kernel.
struct IgemmFixed { int HF, WF, DC; };
constexpr IgemmFixed IGEMM_FIXED[] = {{0, 0, 0}, {3, 3, 8}, {1, 1, 32}, {5, 5, 4}};
constexpr int IGEMM_N_FIXED = 4;
constexpr IgemmFixed IGEMM_WINO = {4, 3, 8};      // the WINO kernels: four row combinations x three columns, 8 channels per unit

// exact number of slab columns the worst pixel tile needs
inline int slab_columns(const ConvView &v, int TI, int TQ, int Wp) {
    const int64_t QN = (int64_t)TI * v.Wo * v.N;
    int best = 0;
    for (int64_t q0 = 0; q0 < QN; q0 += TQ) {
        int64_t qe = q0 + TQ < QN ? q0 + TQ : QN;
        int64_t c0 = q0 / TI, c1 = (qe - 1) / TI;
        int64_t n0 = c0 / v.Wo, n1 = c1 / v.Wo;
        int64_t u0 = (c0 - n0 * v.Wo) * v.Sw;
        int64_t ul = (c1 - n1 * v.Wo) * v.Sw + (n1 - n0) * Wp + v.Wf - 1;
        int sc = (int)(ul - u0 + 1);
        if (sc > best) best = sc;
    }
    return best;
}

// How a tile's reduction is cut into units.  Returns false if nothing fits.
struct UnitCut { int pair_mode, DC, TC, NTR, NS; };

inline bool cut_units(const ConvView &v, int TK, int64_t CP, size_t lds_left, UnitCut *uc) {
    const int T = v.Hf * v.Wf;
    double best = 1e30;
    bool found = false;
    for (int mode = 0; mode < 2; ++mode) {
        for (int NTR = 1; NTR <= T; ++NTR) {
            int TC = (T + NTR - 1) / NTR;
            if (mode == 1) TC += TC & 1;                         // tap pairs: even capacity
            if ((int64_t)(NTR - 1) * TC >= T) continue;          // an empty last range
            for (int DC = 1; DC <= 64; ++DC) {
                if (mode == 0 && (DC & 1)) continue;
                if (DC > 1 && DC - (mode == 0 ? 2 : 1) >= v.Cg) break;   // more padding channels than needed
                int NS = mode == 0 ? (DC / 2) * TC : DC * (TC / 2);
                NS += NS & 1;
                if (NS > 80) continue;
                const size_t lds = (2 * ((size_t)NS * 2 * TK + 255) + 2 * (size_t)DC * CP) * 4;
                if (lds > lds_left) continue;
                // work actually issued per tile / useful work
                const int NCG = (v.Cg + DC - 1) / DC;
                const double issued = (double)NCG * NTR * NS * 2;
                const double useful = (double)v.Cg * T;
                // prefer little padding, then ~40 steps per unit, then few slab reloads (NTR small)
                const double score = issued / useful * (1.0 + 0.002 * (NS > 40 ? NS - 40 : 40 - NS)) *
                                     (1.0 + 0.01 * (NTR - 1));
                if (score < best) { best = score; found = true; uc->pair_mode = mode; uc->DC = DC; uc->TC = TC; uc->NTR = NTR; uc->NS = NS; }
            }
        }
    }
    return found;
}

// bf16 kernel: a unit is 16 channels x TC taps, one MFMA step per tap; the fewest tap ranges whose
// double-buffered weights (TC*2*TK 16-byte words) and slab (2*CP words) fit.
inline bool cut_units_bf16(const ConvView &v, int TK, int64_t CP, size_t lds_left, UnitCut *uc, int planes = 1) {
    const int T = v.Hf * v.Wf;
    for (int NTR = 1; NTR <= T; ++NTR) {
        const int TC = (T + NTR - 1) / NTR;
        if ((int64_t)(NTR - 1) * TC >= T) continue;
        // three planes: the weights do not pass through LDS
        const size_t lds = planes == 3 ? SPLIT_SLABS * 2 * (size_t)CP * 16 * planes
                                       : 2 * ((size_t)TC * 2 * TK + 2 * (size_t)CP) * 16 * planes;
        if (lds > lds_left) continue;
        uc->pair_mode = 0; uc->DC = BF_DC; uc->TC = TC; uc->NTR = NTR; uc->NS = TC;
        return true;
    }
    return false;
}

// Three-plane kernel: block shapes (computing waves WK x WP of MK x MP tiles each), tried in turn.
struct SplitShape { int shape, WK, WP, MK, MP; };
constexpr SplitShape SPLIT_SHAPES[] = {{IG_S64x256, 2, 4, 1, 2}, {IG_S128x128, 4, 2, 1, 2}, {IG_S128x64, 4, 2, 1, 1}, {IG_32x256, 1, 8, 1, 1}};
constexpr int SPLIT_N_SHAPES = 4;

// Estimated time of a three-plane plan in microseconds, and the schedule it is estimated for: `own` whole tiles per block,
// the rest shared.  Cycles of a step: its MFMAs (32 each, WK*WP/4 waves per SIMD), its LDS reads (128 bytes a cycle for
// the block) or its weights' way through the L1 (64 bytes a cycle), whichever is longest, a unit's barrier, a tile's set-up and write-out; the fix-up pass as a launch plus its
// traffic.  Either every block gets the same number of units (left-over tiles shared, fix-up pass), or whole tiles only
// (up to a handful shared, so that the number of blocks stays a multiple of 8).
struct SplitSchedule { int nblocks, own; double us; };
inline SplitSchedule split_schedule(int64_t tiles, int NU, int NS, int64_t slab_bytes, const SplitShape &S, int n_cu, int rows, bool grouped) {
    const double ghz = 2.2;
    const int TK = S.WK * S.MK * 32, TQ = S.WP * S.MP * 32 * rows, waves = S.WK * S.WP;      // TQ: results per filter
    const double mfma = S.MK * S.MP * 6 * 32.0 * waves / 4, lds = waves * 3072.0 * S.MP / 128, l1 = waves * 3072.0 * S.MK / 64;
    double step = mfma;
    if (step < 1.2 * lds) step = 1.2 * lds;
    if (step < 1.2 * l1) step = 1.2 * l1;
    // bytes that a unit brings into the compute unit, at about 40 a cycle
    const double fetch = ((double)NS * 3 * 2 * TK * 16 + (double)slab_bytes) / 40.0;
    double unit = NS * step * 1.15 + 200.0;
    if (unit < fetch) unit = fetch;
    const double tile_over = 2000.0 + TK * TQ * 4.0 / 32.0;
    const double tile_us = (NU * unit + tile_over) / ghz * 1e-3;
    SplitSchedule a, b;
    const int64_t total = tiles * NU;
    a.nblocks = (int)(total < n_cu ? total : n_cu);
    a.own = (int)(tiles / a.nblocks);
    const int64_t left = tiles - (int64_t)a.own * a.nblocks;
    a.us = (double)tiles * tile_us / a.nblocks + (left ? 6.0 + (double)a.nblocks * TK * TQ * 8.0 / 4.0e6 + tile_over / ghz * 1e-3 : 0.0);
    b.own = (int)((tiles + n_cu - 1) / n_cu);
    b.nblocks = (int)(tiles / b.own);
    // 1x1 filters: their tiles are short, and a few left over cost more than what blocks of one XCD share (24x40x344, 1x1x144x344, five images,
    // dzdx: 225 tiles on 224 blocks 50.8 us, on 225 blocks 18.5)
    if (b.nblocks > 64 && !(grouped && (int64_t)b.own * b.nblocks == tiles)) b.nblocks &= ~7;
    b.us = b.own * tile_us;
    if ((int64_t)b.own * b.nblocks != tiles) b.us += 8.0 + (double)b.nblocks * TK * TQ * 2.0 / 4.0e6;
    return b.us <= a.us ? b : a;
}

// The view as the plain sum sees it; wino: of pairs of output rows.
inline PlainView plain_view(const ConvView &v, bool wino) {
    const int area = v.HfA * v.WfA;
    PlainView V = {};
    V.Hf = wino ? 3 : v.Hf; V.Sh = wino ? 1 : v.Sh; V.Wf = v.Wf; V.Sw = v.Sw;
    if (v.fSh) { V.Hf = v.HfA; V.Wf = v.WfA; V.Sh = v.fSh; V.Sw = v.fSw; }
    if (v.pack_mode == 0 || v.pack_mode == 4) {
        V.wo = 0; V.wg = area * v.DfA * v.Kg; V.wk = area * v.DfA; V.wc = area; V.wi = 1; V.wj = v.HfA;
    } else if (v.pack_mode == 1) {
        V.wo = v.pi + v.pSh * (V.Hf - 1) + v.HfA * (v.pj + v.pSw * (v.Wf - 1));
        V.wg = area * v.DfA * v.Cg; V.wk = area; V.wc = area * v.DfA; V.wi = -v.pSh; V.wj = -v.HfA * v.pSw;
    } else if (v.pack_mode == 2) {
        V.wk = 1; V.wc = v.ldk;
    } else {
        V.HfA = v.HfA; V.WfA = v.WfA; V.DfA = v.DfA; V.B0i = v.B0i; V.B0j = v.B0j;
    }
    return V;
}

// wino: `v` is the stride-2, four-tap view of pairs of output rows (wino_view) and wino_Ho the real number of rows
inline bool plan_igemm_kind(const ConvView &v, int n_cu, IgemmPlan *pl, bool bf16, int fixed, bool two = false,
                            int wino_Ho = 0, int planes = 1, int split = 0) {
    const int T = v.Hf * v.Wf;
    const bool wino = wino_Ho > 0, f23s = wino && planes == 3;
    const IgemmFixed FX = wino ? IGEMM_WINO : IGEMM_FIXED[fixed];
    int shape, WK, WP, MK, MP;
    // `two`: blocks of four waves, two of them resident per compute unit (half the LDS each): while one is
    // at its barrier or writes a tile, the other keeps the matrix cores busy
    const size_t lds_limit = two ? IGEMM_LDS_LIMIT / 2 : IGEMM_LDS_LIMIT;
    const int resident = two ? 2 * n_cu : n_cu;
    const SplitShape &SS = SPLIT_SHAPES[split];
    if (planes == 3) { shape = SS.shape; WK = SS.WK; WP = SS.WP; MK = SS.MK; MP = SS.MP; }
    else if (wino && v.Kg > 64) { shape = IG_W128x128; WK = 2; WP = 4; MK = 2; MP = 1; }
    else if (wino) { shape = IG_W64x256; WK = 1; WP = 8; MK = 2; MP = 1; }
    else if (two && v.Kg > 32) { shape = IG_64x256; WK = 1; WP = 4; MK = 2; MP = 2; }
    else if (!bf16 && v.Kg > 64 && v.Kg <= 96) { shape = IG_96x256; WK = 1; WP = 8; MK = 3; MP = 1; }
    else if (v.Kg > 64) { shape = IG_128x256; WK = 2; WP = 4; MK = 2; MP = 2; }
    else if (v.Kg > 32) { shape = IG_64x512; WK = 1; WP = 8; MK = 2; MP = 2; }
    else { shape = IG_32x256; WK = 1; WP = 4; MK = 1; MP = 2; }
    const int TK = WK * MK * 32, TQ = WP * MP * 32, NT = 64 * WK * WP;
    // threads of the fetching (bf16: staging) waves
    const int NL = 64 * (planes == 3 ? SPLIT_STAGE_WAVES : IGEMM_LOADER_WAVES);
    const int Wp = (v.Wo - 1) * v.Sw + v.Wf;
    // 1x1 filters in three planes: 16-channel groups per unit, as many as the slab holds, shared out evenly
    const bool grouped = planes == 3 && T == 1;
    int GR = 1;
    if (grouped) {
        const int groups = (v.Cg + BF_DC - 1) / BF_DC, most = split_samples(false) / TQ, units = (groups + most - 1) / most;
        GR = (groups + units - 1) / units;
    }
    // candidates for the row-block height
    int cand[48];
    int nc = 0;
    cand[nc++] = v.Ho;
    for (int parts = 2; parts <= 16; ++parts) cand[nc++] = (v.Ho + parts - 1) / parts;
    for (int t = 32; t <= 256; t += 32) cand[nc++] = t;
    for (int t = 1; t <= 16; t *= 2) cand[nc++] = t;
    if (grouped) nc = 1;               // no slab rows: whole columns
    const bool input_streams = 4.0 * v.H * v.W * (double)v.Ctot * v.N > 32.0 * 1024 * 1024;
    double best_score = 1e30;
    int bestTI = 0, bestSC = 0;
    UnitCut best_uc = {};
    for (int a = 0; a < nc; ++a) {
        const int TI = cand[a];
        if (TI < 1 || TI > v.Ho) continue;
        const int64_t SR = f23s ? TI : (int64_t)(TI - 1) * v.Sh + v.Hf;     // row combinations: one slab sample per pair
        if (SR > 8192 && !grouped) continue;
        if ((int64_t)TI * v.Wo * v.N >= ((int64_t)1 << 30)) continue;
        const int SC = slab_columns(v, TI, TQ, Wp);
        const int64_t CP = grouped ? (int64_t)GR * TQ : (SR * SC + 63) / 64 * 64;
        if (CP > (planes == 3 ? split_samples(f23s) : (bf16 ? bf_ept_max(NL) : 32) * NL)) continue;
        // an image crossing inside a tile moves the window by whole images: keep offsets in range
        const int64_t span = (int64_t)SC / Wp + 2;
        if ((double)span * v.Ctot * v.H * v.W * 4.0 >= 2147483647.0) continue;
        if ((double)(span + 1) * v.Ktot * v.OH * v.OW * 4.0 >= 2147483647.0) continue;   // and inside its output window
        const int EPT = (int)((CP + NL - 1) / NL);
        const size_t fixed_lds = ((planes == 3 ? 0 : (size_t)EPT * NL) + (planes == 3 ? (v.mD ? 3 : 1) * SPLIT_BIASES : 2) * TK + 4) * 4;
        UnitCut uc;
        if (f23s) {
            uc.pair_mode = 0; uc.DC = BF_DC; uc.TC = 3; uc.NTR = 1; uc.NS = 3;
            if (fixed_lds + 64 + SPLIT_SLABS * 6 * (size_t)CP * 16 > lds_limit) continue;
        } else if (bf16) {
            if (fixed_lds + 64 > lds_limit) continue;
            if (!cut_units_bf16(v, TK, CP, lds_limit - fixed_lds - 64, &uc, planes)) continue;
            if (grouped) { uc.DC = BF_DC * GR; uc.NS = GR; }
        } else if (fixed || wino) {
            uc.pair_mode = 0; uc.DC = FX.DC; uc.TC = T; uc.NTR = 1; uc.NS = (FX.DC / 2) * T;
            if ((2 * ((size_t)uc.NS * 2 * TK + 255) + 2 * (size_t)uc.DC * CP) * 4 + fixed_lds > lds_limit) continue;
        } else {
            if (fixed_lds + 4096 + 16384 > lds_limit) continue;
            // the offset table needs NTR*NS*2 ints: reserve 16 KB for it up front
            if (!cut_units(v, TK, CP, lds_limit - fixed_lds - 16384, &uc)) continue;
            if ((size_t)uc.NTR * uc.NS * 2 * 4 > 16384) continue;
        }
        const int RB = (v.Ho + TI - 1) / TI;
        const int64_t QN = (int64_t)TI * v.Wo * v.N;
        const int64_t PT = (QN + TQ - 1) / TQ;
        // rows of pixel tiles and of filter tiles that compute nothing
        const double mfma_waste = (double)RB * PT * TQ / ((double)v.Ho * v.Wo * v.N) *
                                  (double)((v.Kg + TK - 1) / TK * TK) / (double)v.Kg;
        const int NCG = (v.Cg + uc.DC - 1) / uc.DC * (f23s ? 4 : 1);
        const double red_waste = (double)NCG * uc.NTR * uc.NS * (bf16 ? BF_DC : 2) / ((double)v.Cg * T);
        // when the input streams from memory, short slab rows waste most of every 128-byte line they touch
        // results are stored in column runs of TI samples: short runs are partial memory lines
        double score = mfma_waste * red_waste * (1.0 + 0.05 * (double)CP / TQ) *
                       (input_streams ? 1.0 + 4.0 / (double)SR : 1.0) * (1.0 + 2.0 / (double)TI);
        // bf16 kernels: every tap range of a group of channels is a unit of its own (a barrier, a prologue of LDS
        // reads); a smaller slab that leaves room for more taps per unit is worth a less regular row block
        // (measured with split operands, same box: layer 4a with one tap range 0.41 against 0.50 ms with three;
        // 4b with two 0.378 against 0.40 with three)
        if (bf16) score *= 1.0 + 0.5 * (uc.NTR - 1);
        if (planes == 3)     // microseconds; short slab rows and short column runs of results as above
            score = split_schedule((int64_t)v.G * RB * PT * ((v.Kg + TK - 1) / TK), NCG * uc.NTR, uc.NS, CP * (f23s ? 128 : 64), SS, n_cu, f23s ? 2 : 1, grouped).us *
                    (input_streams ? 1.0 + 1.0 / (double)SR : 1.0) * (1.0 + 0.5 / (double)TI);
        if (wino && !f23s) {
            // The row-pair kernels issue fewer MFMAs per staged byte and per stored line, and what was measured on
            // them weighs differently: short slab rows cost little, column runs of results (2*TI samples) that are
            // whole 128-byte lines are worth some 5 % (layer 4a: 32-row runs 0.74 ms, 112-row runs 0.78, 28-row 0.80).
            const double run_bytes = 8.0 * TI;
            const bool whole_lines = (8 * TI) % 128 == 0 && ((int64_t)v.OH * 4) % 128 == 0;
            score = mfma_waste * red_waste * (1.0 + 0.05 * (double)CP / TQ) *
                    (input_streams ? 1.0 + 1.0 / (double)SR : 1.0) * (1.0 + (whole_lines ? 0.0 : 0.25 * 128.0 / run_bytes));
        }
        if (score < best_score) { best_score = score; bestTI = TI; bestSC = SC; best_uc = uc; }
    }
    if (!bestTI) return false;

    IgemmParams &P = pl->P;
    P = IgemmParams{};
    P.H = v.H; P.W = v.W; P.N = v.N; P.Ctot = v.Ctot; P.Cg = v.Cg;
    P.Ho = v.Ho; P.Wo = v.Wo; P.Ktot = v.Ktot; P.Kg = v.Kg; P.G = v.G;
    P.Hf = v.Hf; P.Wf = v.Wf; P.Sh = v.Sh; P.Sw = v.Sw; P.Pt = v.Pt; P.Pl = v.Pl;
    P.TI = bestTI; P.RB = (v.Ho + bestTI - 1) / bestTI;
    P.Wp = Wp;
    P.SR = f23s ? bestTI : (bestTI - 1) * v.Sh + v.Hf; P.SRP = P.SR;
    P.CP = grouped ? GR * TQ : (P.SRP * bestSC + 63) / 64 * 64;
    P.EPT = (P.CP + NL - 1) / NL;
    P.KT = (v.Kg + TK - 1) / TK;
    P.QN = bestTI * v.Wo * v.N;
    P.PT = (P.QN + TQ - 1) / TQ;
    P.DC = best_uc.DC; P.TC = best_uc.TC; P.NTR = best_uc.NTR; P.NS = best_uc.NS; P.pair_mode = best_uc.pair_mode;
    P.NU = ((v.Cg + P.DC - 1) / P.DC) * P.NTR * (f23s ? 4 : 1);
    const int64_t tiles = (int64_t)v.G * P.RB * P.PT * P.KT;
    if (tiles >= ((int64_t)1 << 30)) return false;
    P.tiles = (int)tiles;
    const int64_t total = tiles * P.NU;
    P.nblocks = (int)(total < resident ? total : resident);
    // whole tiles first, one share of the left-over tiles after (see IgemmParams::own): fewer tiles go through
    // the workspace and the fix-up pass than when everything is shared
    P.own = (int)(tiles / P.nblocks);
    if (planes == 3) {
        const SplitSchedule sc = split_schedule(tiles, P.NU, P.NS, (int64_t)P.CP * (f23s ? 128 : 64), SS, n_cu, f23s ? 2 : 1, grouped);
        P.nblocks = sc.nblocks;
        P.own = sc.own;
        // Row pairs: a tile in at most 32 pieces.  With 64 or more the fix-up pass, which adds them one after another, costs more
        // than the shorter pieces save (14x13x256, 96 filters, two images: 34.1 us on 256 blocks, 29.0 on 128; 7x7x512 -> 512, one
        // image 43.3 and 38.0; 16 pieces at most: 26.3 and 38.1, but 7x9x309, 336 filters, four images 37.9 against 35.7).
        if (f23s && P.own == 0 && P.nblocks > 32 * (int)tiles) P.nblocks = 32 * (int)tiles;
    } else if (!bf16 && 2 * tiles >= resident && tiles < resident) {
        // Somewhat fewer tiles than compute units: sharing every tile keeps all units busy but sends every tile through
        // the workspace and the fix-up pass; one whole tile per block leaves some units idle and needs neither.
        // Times in microseconds: a unit's MFMAs at about 80 % of the matrix core's rate (two waves per SIMD with
        // 512 threads or two resident blocks), the fix-up as a launch plus its traffic at about 4 TB/s.
        const double unit_us = (two ? 2 : NT / 256) * (double)P.NS * MK * MP * 64.0 / 0.8 / 2400.0;
        const double fix_us = 6.0 + (double)P.nblocks * TK * TQ * (wino ? 16.0 : 8.0) / 4.0e6;
        const double shared_us = (double)((total + P.nblocks - 1) / P.nblocks) * unit_us + fix_us;
        if ((double)P.NU * unit_us <= shared_us) {
            P.nblocks = (int)tiles;
            P.own = 1;
        }
    }
    // two blocks per compute unit, whole tiles for every block and some left over: the blocks dispatched
    // first take the left-over units (see IgemmParams::nshare)
    P.nshare = P.nblocks;
    if (two && P.own >= 1 && (int64_t)P.own * P.nblocks != tiles && P.nblocks == resident && P.nblocks % 16 == 0)
        P.nshare = P.nblocks / 2;
    P.walk = make_sk_walk((tiles - (int64_t)P.own * P.nblocks) * (P.NU / (planes == 3 && wino_Ho ? 4 : 1)), P.nshare, P.NU);
    P.OH = v.OH; P.OW = v.OW; P.oi0 = v.oi0; P.osi = v.osi; P.oj0 = v.oj0; P.osj = v.osj;
    P.mD = v.mD; P.mPt = v.mPt; P.mPl = v.mPl;
    P.wino_Ho = wino_Ho;
    if (bf16 && planes < 3 && v.pack_mode == 2) return false;       // the fully-connected views compute in fp32
    pl->F.VC = v.Cg;
    pl->F.fSh = pl->F.fSw = 0;
    if (v.fSh) {
        P.Cg = v.Cg / (v.fSh * v.fSw);
        pl->F.fSh = v.fSh; pl->F.fSw = v.fSw; pl->F.dfSh = make_div32(v.fSh); pl->F.dfSS = make_div32(v.fSh * v.fSw);
    }
    if (planes == 3) pl->V = plain_view(v, wino);
    P.dTI = make_div32(P.TI); P.dWo = make_div32(P.Wo); P.dWp = make_div32(P.Wp); P.dSRP = make_div32(P.SRP);
    P.dKT = make_div32(P.KT); P.dRB = make_div32(P.RB); P.dPT = make_div32(P.PT);
    // packed weights per unit, in 32-bit words: bf16 steps hold 2 octets x TK filters x 16 bytes
    const size_t wsz = bf16 ? (size_t)P.NS * planes * 2 * TK * 4 : ((size_t)P.NS * 2 * TK + 255) / 256 * 256;
    P.WSZ = (int)wsz;
    pl->packed_floats = (size_t)v.G * P.KT * P.NU * wsz;
    if (pl->packed_floats * 4 >= 2147483647ull) return false;
    P.packed_bytes = (unsigned)(pl->packed_floats * 4);
    // no workspace for partial tiles when no tile is shared
    pl->partial_floats = P.nblocks > 1 && (int64_t)P.own * P.nblocks != tiles ? (size_t)2 * P.nblocks * TK * TQ * (wino ? 2 : 1) : 0;
    pl->shape = shape; pl->bf16 = bf16; pl->planes = bf16 ? planes : 1; pl->fixed = fixed; pl->TK = TK; pl->TQ = TQ; pl->NT = NT;
    pl->score = best_score;
    if (planes == 3)
        pl->lds_bytes = ((size_t)(v.mD ? 3 : 1) * SPLIT_BIASES * TK + (size_t)SPLIT_SLABS * 6 * P.CP * 4 + 4) * sizeof(float);
    else if (bf16)
        pl->lds_bytes = (2 * wsz + 2 * (size_t)planes * 2 * P.CP * 4 + (size_t)P.EPT * NL + 2 * TK + 4) *
                        sizeof(float);
    else
        pl->lds_bytes = (2 * wsz + 2 * (size_t)P.DC * P.CP + (size_t)P.EPT * NL + 2 * TK +
                         (fixed || wino ? 0 : (size_t)P.NTR * P.NS * 2) + 4) * sizeof(float);
    if (pl->lds_bytes > lds_limit) return false;

    PackParams &Q = pl->Q;
    Q = PackParams{};
    Q.Hf = v.Hf; Q.Wf = v.Wf; Q.HfA = v.HfA; Q.WfA = v.WfA; Q.DfA = v.DfA;
    Q.Kg = v.Kg; Q.Cg = v.Cg; Q.G = v.G; Q.KT = P.KT; Q.NU = P.NU; Q.NTR = P.NTR; Q.NS = P.NS; Q.WSZ = P.WSZ; Q.TK = TK; Q.MK = MK;
    Q.DC = P.DC; Q.TC = P.TC; Q.pair_mode = P.pair_mode; Q.mode = v.pack_mode;
    Q.Sh = v.pSh; Q.Sw = v.pSw; Q.pi = v.pi; Q.pj = v.pj; Q.ldk = v.ldk;
    if (v.fSh) { Q.Sh = v.fSh; Q.Sw = v.fSw; }
    Q.mD = v.mD; Q.Pt = v.mPt; Q.Pl = v.mPl; Q.B0i = v.B0i; Q.B0j = v.B0j;
    Q.wino = wino ? 1 : 0;
    Q.planes = bf16 ? planes : 1;
    Q.total = (int)pl->packed_floats;
    if (grouped) { Q.NU *= GR; Q.NS = 1; Q.WSZ /= GR; }       // groups follow one another in memory, as units of one
    return true;
}

// 3x3 filters at stride 1 with at least 16 channels per group: the view of pairs of output rows that the
// WINO kernels compute (kern_igemm.h).  Its rows are pairs, its four "taps" per column the four input rows a
// pair reads; results go to rows oi0 + osi * (2 * pair + {0, 1}) of the output array.
inline bool wino_view(const ConvView &v, ConvView *out) {
    if (v.Hf != 3 || v.Wf != 3 || v.Sh != 1 || v.Sw != 1 || v.mD || v.pack_mode > 1) return false;
    if (v.HfA != 3 || v.WfA != 3 || (v.pack_mode == 1 && (v.pSh != 1 || v.pSw != 1))) return false;
    if (v.Cg < 2 * IGEMM_WINO.DC || v.Ho < 2) return false;      // channels are padded to units of 8 (zero weights, slab reads as zero)
    if (v.Kg <= 32) return false;      // the WINO tiles are 64 or 128 filters wide; narrower layers keep the 32-filter tiles
    ConvView p = v;
    p.Hf = 4; p.Sh = 2; p.Ho = (v.Ho + 1) / 2; p.osi = 2 * v.osi;
    *out = p;
    return true;
}
inline bool wino_enabled() {
    // process-wide override for benchmarks; a caller chooses per call with MCN_PREC_FP32_PLAIN
    static const bool off = getenv("MCN_NO_WINO") != nullptr;
    return !off;
}

// Views the three-plane kernel (kern_igemm_split.h) can take.  1x1 filters (fully-connected layers' products among them) in units of several
// groups of 16 channels: with one, a unit was one step (768 cycles of MFMAs), and its staging (loads, split, barrier) took longer (28x28x512,
// 1x1x512x128, 64 images: forward 93 us, now 60, 83 on the fp32 kernel).  Not merged phases of them.
inline bool split_possible(const ConvView &v) {
    return v.Cg >= BF_DC && (!v.mD || v.Hf * v.Wf >= 2);
}

// Row pairs in three planes (F23): deep layers whose plane and batch give at most as many tiles of 128 filters x 64 pairs as
// there are compute units.
inline bool split_pairs_possible(const ConvView &pv, int n_cu) {
    const int64_t tiles = (((int64_t)pv.Ho * pv.Wo * pv.N + 127) / 128) * ((pv.Kg + 127) / 128) * pv.G;
    return pv.Cg >= 256 && pv.Kg > 64 && 2 * tiles <= n_cu;
}

// Estimated microseconds of a whole call (packing, main kernel, fix-up pass), for the choice between the two kernels only.  The
// constants are a fit to 568 forward and dzdx calls of random layers on 256 compute units, both kernels timed in turn (5 to 230
// samples a side, 1 to 128 images, 8 to 384 channels and filters, 2 to 121 taps, strides 1 to 4): the estimate is off by 9 %
// (three planes) and 16 % (fp32) of a call, 1 standard deviation.
inline double call_us(const ConvView &v, const IgemmPlan &pl, int n_cu) {
    const IgemmParams &P = pl.P;
    const double out_mb = 4e-6 * v.Ho * v.Wo * (double)v.Kg * v.G * v.N, pack_mb = 4e-6 * (double)pl.packed_floats;
    const int64_t left = P.tiles - (int64_t)P.own * P.nblocks;         // tiles that are shared
    const double shared = left ? (double)((left * P.NU + P.nblocks - 1) / P.nblocks) : 0.0;      // units of them per block
    const double part_mb = left && P.NU > 1 ? 4e-6 * (double)pl.partial_floats : 0.0;
    if (pl.planes == 3) {
        const double step = pl.shape == IG_32x256 ? 0.25 : pl.shape == IG_S64x256 ? 0.42 : pl.shape == IG_S128x128 ? 0.44 : 0.265;
        const double unit = 0.70 + P.NS * step;
        return 10.7 + 0.95 * pack_mb + P.own * P.NU * unit + (left ? 4.7 + shared * unit + 0.29 * part_mb : 0.0) + 0.37 * out_mb;
    }
    const int resident = (P.nblocks + n_cu - 1) / n_cu;                // blocks that share a compute unit
    const double mfma_us = pl.TK * pl.TQ / 1024 / 4.0 * P.NS * 64.0 / 2400.0;      // a unit's MFMAs at full rate
    const double slow = pl.shape == IG_64x512 ? 1.31 : pl.shape == IG_32x256 ? 0.92 : pl.shape == IG_64x256 ? 0.89 : pl.shape == IG_96x256 ? 1.10 : 0.98;
    const double unit = resident * (0.64 + mfma_us * slow);
    return 10.4 + 2.8 * pack_mb + P.own * P.NU * unit + (left ? 3.5 + shared * unit + 0.22 * part_mb : 0.0) + 0.126 * out_mb;
}

// Whether the three-plane kernel is the faster one for view v; split, fp32: the two plans.
// Over those 568 calls: always three planes 27.8 ms, always fp32 36.4 ms, by this rule 27.55 ms, the faster of the two each time
// 27.1 ms.  Small layers are what it keeps on the fp32 kernel, which cuts a tile's reduction finer: 32x32x32 -> 3, 5x5,
// eight images 16.4 us against 25.1, 16x16x32, 5x5x32x32, one image 15.3 against 25.6.
// Row pairs, whose slab the planner keeps within 128 samples (split_samples), always: of 222 calls one is slower than on the fp32
// kernel by more than 1 % (52x52x424, 121 filters, nine images 145 -> 149 us), half of them by 14 % or more faster.  With slabs of up to 256
// samples beside the 64 pairs, staging bound them (58x58x280, 160 filters, three images 91 -> 111 us).
// 1x1 filters (49 random layers, 98 calls): always fp32 3.11 ms, by this rule 2.49; products of 31 fully-connected layers (62 calls) 2.84 and 2.02;
// none of either that it sends here is slower by more than 2 %.
inline bool split_faster(const ConvView &v, const IgemmPlan &split, const IgemmPlan &fp32, int n_cu) {
    if (split.P.wino_Ho) return true;
    return call_us(v, split, n_cu) < 0.97 * call_us(v, fp32, n_cu);
}

// The instantiation with this view's filter size if there is one, its channels divide into the
// fixed units and a plan fits; the general kernel otherwise.
// row_pairs: 3x3 stride-1 views may take the kernels that compute two output rows from four products per
// filter column (the caller asks for the plain order of summation with MCN_PREC_FP32_PLAIN).
// planes (bf16 only): 2 = split operands (kern_igemm_bf16.h)
inline bool plan_igemm(const ConvView &v, int n_cu, IgemmPlan *pl, bool bf16 = false, bool row_pairs = true, int planes = 1) {
    if (bf16 && planes == 3) {
        bool ok = false;
        ConvView pv;
        const bool pairs = wino_enabled() && wino_view(v, &pv);
        if (pairs && !split_pairs_possible(pv, n_cu)) return false;
        for (int f = 0; f < SPLIT_N_SHAPES; ++f) {
            const int TK = SPLIT_SHAPES[f].WK * SPLIT_SHAPES[f].MK * 32;
            if (TK == 32 ? v.Kg > 32 : v.Kg <= TK / 2) continue;      // half of the tile would be empty
            if (pairs && SPLIT_SHAPES[f].shape != IG_S128x64) continue;     // three sums and two rows per pair: registers for no larger tile
            IgemmPlan one;
            if (plan_igemm_kind(pairs ? pv : v, n_cu, &one, true, 0, false, pairs ? v.Ho : 0, 3, f) && (!ok || one.score < pl->score)) { *pl = one; ok = true; }
        }
        return ok;
    }
    if (bf16) return plan_igemm_kind(v, n_cu, pl, true, 0, false, 0, planes);
    ConvView pv;
    if (row_pairs && wino_enabled() && wino_view(v, &pv) && plan_igemm_kind(pv, n_cu, pl, false, 0, false, v.Ho)) return true;
    // the instantiation with this view's filter size, if there is one and the channels divide into its units
    int fixed = 0;
    for (int f = 1; f < IGEMM_N_FIXED; ++f) {
        const IgemmFixed FX = IGEMM_FIXED[f];
        if (v.Hf == FX.HF && v.Wf == FX.WF && v.Cg >= 2 * FX.DC && v.Cg % FX.DC == 0) fixed = f;
    }
    for (int f = fixed;; f = 0) {
        // With more than 32 filters per group: two resident blocks of four waves rather than one of eight,
        // unless half the LDS forces a much worse row-block height on it (the scores are comparable).
        // Up to 32 filters the block has four computing waves either way; two of them per compute unit pay when
        // there are more tiles than compute units (layer 2a, 400 tiles: every block one whole tile, no fix-up
        // pass, forward 20 -> 17 us), not when tiles are shared anyway (layer 2b, 100 tiles in 512 pieces: +23 %).
        IgemmPlan one, two;
        const bool ok1 = plan_igemm_kind(v, n_cu, &one, false, f);
        bool ok2 = plan_igemm_kind(v, n_cu, &two, false, f, true);
        if (ok2 && v.Kg <= 32 && two.P.tiles <= n_cu) ok2 = false;
        if (ok2 && (!ok1 || two.score <= 1.15 * one.score)) { *pl = two; return true; }
        if (ok1) { *pl = one; return true; }
        if (f == 0) return false;
    }
}

}  // namespace mcn

// ---- filter derivative (kern_wgrad.h) ---------------------------------------------------
#include "kern_wgrad.h"
namespace mcn {

// WG_W*: the WINO kernels (filters x (filter column, channel) pairs)
// WG_96x128, WG_96x384: 65 to 96 filters per group; the second on 12 computing waves, for filters of more than 256
// coefficients per group (one tile then holds 384 of them and dzdy is staged once for all)
enum WgradShape { WG_128x128 = 0, WG_64x192 = 1, WG_32x256 = 2, WG_W128x128 = 3, WG_W64x192 = 4, WG_96x128 = 5, WG_96x384 = 6 };

struct WgradPlan {
    int shape;
    int TK, TR, NT;
    WgradParams P;
    size_t lds_bytes;
    int occupancy;           // resident blocks per compute unit
    size_t partial_floats;   // 2 slots of TK*TR per resident block
    bool wino;               // kern_wgrad.h, template flag WINO; TR then counts coefficients (3 per B lane)
};

// wino: the WINO kernels (3x3 filters at stride 1, more than 32 filters per group): tiles of 128 filters x 128
// (filter column, channel) pairs on 8 computing waves, or, up to 64 filters per group, 64 x 192 on 12 computing
// waves (one 32 x 32 tile with its four sets of accumulators each), which holds all of a 64-channel layer.
inline bool plan_wgrad(const ConvView &v, int n_cu, WgradPlan *pl, bool wino = false) {
    if (wino && (v.Hf != 3 || v.Wf != 3 || v.Sh != 1 || v.Sw != 1 || v.Ho < 2 || v.Kg <= 32)) return false;
    // A filter row that meets no input row at all (planes of one or two rows under large pads) has a derivative of
    // exactly zero; the WINO kernel would form it as a difference of sums that cancel only up to rounding.
    if (wino && (v.H + v.Pt < 3 || v.Ho - 1 < v.Pt)) return false;
    // Each of its sums also holds the products of the neighbouring row of dzdy, which cancel up to rounding; over a
    // handful of terms one small factor can leave that rounding large against the result's own terms.
    if (wino && (int64_t)v.N * v.Ho * v.Wo < 64) return false;
    const int T = wino ? v.Wf : v.Hf * v.Wf;             // B lanes per channel
    if ((int64_t)v.Hf * v.Wf * v.Cg >= ((int64_t)1 << 30)) return false;
    const int R = T * v.Cg;                              // B lanes in all
    // byte offsets into x and dzdy are 32-bit and relative to the start of an image
    if ((double)v.H * v.W * v.Ctot * 4 >= 2147483647.0) return false;
    if ((double)v.Ho * v.Wo * v.Ktot * 4 >= 2147483647.0) return false;
    int shape, WK, WR, MK, MR;
    if (wino && v.Kg > 64) { shape = WG_W128x128; WK = 2; WR = 4; MK = 2; MR = 1; }
    else if (wino) { shape = WG_W64x192; WK = 2; WR = 6; MK = 1; MR = 1; }     // 12 computing waves, one tile each per set
    else if (v.Kg > 64 && v.Kg <= 96 && R > 256) { shape = WG_96x384; WK = 3; WR = 4; MK = 1; MR = 3; }
    else if (v.Kg > 64 && v.Kg <= 96) { shape = WG_96x128; WK = 1; WR = 4; MK = 3; MR = 1; }
    else if (v.Kg > 64) { shape = WG_128x128; WK = 2; WR = 2; MK = 2; MR = 2; }
    else if (v.Kg > 32) { shape = WG_64x192; WK = 2; WR = 2; MK = 1; MR = 3; }
    else { shape = WG_32x256; WK = 1; WR = 4; MK = 1; MR = 2; }
    const int TK = WK * MK * 32, TR = WR * MR * 32, NT = 64 * WK * WR;
    const int RT = (R + TR - 1) / TR;
    int nch_max = 0;
    for (int rt = 0; rt < RT; ++rt) {
        const int lo = rt * TR, hi = (lo + TR < R ? lo + TR : R);
        const int n = (hi - 1) / T - lo / T + 1;
        if (n > nch_max) nch_max = n;
    }
    const int klim = v.Kg < TK ? v.Kg : TK;

    // a unit is a patch of TI rows x MC columns of one image's output plane, at most 128 pixels
    double best = 1e30;
    int bestTI = 0, bestMC = 0, bestSRP = 0, bestCP = 0, bestOcc = 0, bestPCHP = 0;
    size_t bestLds = 0;
    for (int TI = 1; TI <= v.Ho && TI <= 128; ++TI) {
        const int RB = (v.Ho + TI - 1) / TI;
        if (TI > 1 && TI < v.Ho && (v.Ho + TI - 2) / (TI - 1) == RB) continue;   // a smaller TI gives the same row blocks
        const int TIE = wino ? (TI + 3) & ~3 : (TI + 1) & ~1;
        const int64_t SR = (int64_t)(TIE - 1) * v.Sh + v.Hf;     // rows the padding pixel of an odd TI reads are staged too
        if (SR > 16384) continue;
        // pitches chosen so that the 32 coefficients a half-wave reads fall in 32 different LDS banks:
        // bank(r) = fi + SRP*fj + CP*c  ==  r  (mod 32)
        // (WINO: 8-byte reads at SRP/2 * fj + CP/2 * c, in units of 8 bytes: SRP/2 odd and CP = 3 SRP (mod 64)
        // make that SRP/2 * (fj + 3c), different for the lanes of a half-wave)
        int SRP = (int)SR;
        if (wino) while (SRP % 4 != 2) ++SRP;
        else while (SRP % 32 != v.Hf % 32) ++SRP;
        for (int MC = 1; MC <= v.Wo && TIE * MC <= 128; ++MC) {
            const int CC = (v.Wo + MC - 1) / MC;
            if (MC > 1 && MC < v.Wo && (v.Wo + MC - 2) / (MC - 1) == CC) continue;
            const int PCH = TIE * MC;
            const int64_t SC = (int64_t)(MC - 1) * v.Sw + v.Wf;
            if (SC >= 32768) continue;
            int64_t CP = (int64_t)SRP * SC;
            if (wino) while (CP % 64 != (3 * SRP) % 64) ++CP;
            else while (CP % 32 != T % 32) ++CP;
            const int64_t XS = (int64_t)nch_max * CP;
            int PCHP = PCH | 1;
            if (wino) { PCHP = PCH; while (PCHP % 4 != 2) ++PCHP; }
            const int EPT = (int)(((int64_t)SRP * SC + NT - 1) / NT);
            const int64_t lds = (2 * (int64_t)TK * PCHP + 2 * XS + (int64_t)EPT * NT + 4) * 4;
            if (lds > (int64_t)IGEMM_LDS_LIMIT) continue;
            int occ = (int)((int64_t)IGEMM_LDS_LIMIT / lds);
            if (occ > 2) occ = 2;   // the kernels are compiled for two waves per SIMD
            if (NT >= 512) occ = 1; // 8 or 12 computing + 4 fetching waves: one block per compute unit
            // cost of a unit in matrix-core cycles: its MFMAs plus what staging it costs beside them
            // (fitted to measurements: a fixed part and a part per staged element, about twice as
            // much when only one block fits a compute unit and nothing else hides it)
            const double units = (double)v.N * RB * CC;
            const double mfma = wino ? (double)(PCH / 4) * 4 * MK * MR * 64.0 : (double)(PCH / 2) * MK * MR * 64.0;
            const double elems = (double)klim * PCH + (double)nch_max * (double)(SRP * SC);
            // row runs that do not start on 128-byte lines cost extra memory transactions (a patch of whole
            // columns is one contiguous run of dzdy)
            const bool aligned = TI == v.Ho || (TI * 4) % 128 == 0;
            const double ovh = (1700.0 + 0.18 * elems) * (occ >= 2 ? 1.0 : 2.0) * (aligned ? 1.0 : 1.25);
            const double score = units * (mfma + ovh);
            if (score < best) {
                best = score; bestTI = TI; bestMC = MC; bestSRP = SRP; bestCP = (int)CP; bestOcc = occ;
                bestLds = (size_t)lds; bestPCHP = PCHP;
            }
        }
    }
    if (!bestTI) return false;

    WgradParams &P = pl->P;
    P = WgradParams{};
    P.H = v.H; P.W = v.W; P.N = v.N; P.Ctot = v.Ctot; P.Cg = v.Cg;
    P.Ho = v.Ho; P.Wo = v.Wo; P.Ktot = v.Ktot; P.Kg = v.Kg; P.G = v.G;
    P.Hf = v.Hf; P.Wf = v.Wf; P.Sh = v.Sh; P.Sw = v.Sw; P.Pt = v.Pt; P.Pl = v.Pl;
    P.TI = bestTI; P.RB = (v.Ho + bestTI - 1) / bestTI;
    P.MC = bestMC; P.CC = (v.Wo + bestMC - 1) / bestMC;
    P.TIE = wino ? (bestTI + 3) & ~3 : (bestTI + 1) & ~1;
    P.SR = (P.TIE - 1) * v.Sh + v.Hf;
    P.SRP = bestSRP; P.SC = (bestMC - 1) * v.Sw + v.Wf; P.CP = bestCP;
    P.EPT = (bestSRP * P.SC + NT - 1) / NT;
    P.KT = (v.Kg + TK - 1) / TK; P.RT = RT;
    P.PCH = P.TIE * bestMC; P.PCHP = bestPCHP;
    const int64_t NU = (int64_t)v.N * P.RB * P.CC;
    if (NU >= ((int64_t)1 << 30)) return false;
    P.NU = (int)NU;
    P.R = v.Hf * v.Wf * v.Cg;
    P.XS = nch_max * bestCP;
    const int64_t tiles = (int64_t)v.G * P.KT * RT;
    if (tiles >= ((int64_t)1 << 30)) return false;
    P.tiles = (int)tiles;
    const int64_t total = tiles * NU;
    const int64_t want = (int64_t)n_cu * bestOcc;
    P.nblocks = (int)(total < want ? total : want);
    P.nchunks = 0;
    // Arrays that stream from memory: the chunked schedule (kern_wgrad.h) reads them about once instead of
    // once per tile, if it keeps the compute units about as busy as equal ranges would (rounds of `want`
    // resident blocks, each block a chunk plus a fixed part).  It costs about 1 % of time on the large
    // layers (a few idle blocks, chunks that differ by a unit) and saves 2-10x of their memory traffic.
    if (4.0 * ((double)v.H * v.W * v.Ctot + (double)v.Ho * v.Wo * v.Ktot) * v.N > 64.0 * 1024 * 1024) {
        int best_nch = 0;
        double best_time = 1e300;
        for (int64_t nch = 1; nch <= NU && nch * tiles <= 4 * want; ++nch) {
            const int64_t rounds = (nch * tiles + want - 1) / want;
            const double time = (double)rounds * ((double)((NU + nch - 1) / nch) + 2.0);
            if (time < best_time * 0.9999999) { best_time = time; best_nch = (int)nch; }
        }
        if (best_nch > 0 && ((double)total / (double)want) / best_time >= 0.95) {
            P.nchunks = best_nch;
            P.nblocks = (int)(tiles * best_nch);
        }
    }
    // chunk weights (WgradParams::n_first): uneven only when two blocks share each compute unit and every
    // chunk has units to spare
    P.walk = make_sk_walk(P.nchunks > 0 ? NU : total, P.nchunks > 0 ? P.nchunks : P.nblocks, P.NU);
    P.n_first = n_cu; P.w_first = 1; P.w_later = 1;
    if (P.nchunks > 0 && bestOcc == 2 && P.nblocks > n_cu && NU / P.nchunks >= 16) {
        P.w_first = 3; P.w_later = 2;      // measured on layers 4a/4b: 11:9 -1.5 %, 3:2 -2.2 %, 13:7 +1 %
    }
    // one tile, cut into a chunk per block: the blocks of an XCD take the units of their common range in turn
    // (WgradParams::deal; remainders in 32 bits: NU < 2^30 and rem * chunk < nchunks^2)
    P.deal = (P.nchunks >= 16 && P.tiles == 1 && P.nchunks % 8 == 0 && P.w_first == P.w_later && P.nchunks <= 32768) ? 1 : 0;
    pl->occupancy = bestOcc;
    pl->wino = wino;
    pl->partial_floats = P.nblocks > 1 ? (size_t)2 * P.nblocks * TK * TR * (wino ? 3 : 1) : 0;
    pl->shape = shape; pl->TK = TK; pl->TR = wino ? 3 * TR : TR; pl->NT = NT;
    pl->lds_bytes = bestLds;
    return true;
}

}  // namespace mcn

// ---- filter derivative on the bf16 matrix core: fp32 operands in three planes (kern_wgrad_split.h), or rounded to bf16 (kern_wgrad_bf16.h) -----
#include "kern_wgrad_split.h"
#include "kern_wgrad_bf16.h"
namespace mcn {

enum WgradSplitShape { WGS_128x128 = 0, WGS_64x256 = 1, WGS_32x256 = 2, WGB_128x384 = 3, WGB_128x256 = 4, WGB_128x128 = 5, WGB_64x768 = 6, WGB_64x512 = 7, WGB_64x256 = 8 };
// Tiles (filters x coefficients) and how much a staging thread brings per unit (launch_wgrad_split): octets of dzdy and of x; and for LINEAR, 0: no
// such instantiation.
struct WgradSplitTile { int planes, TK, TR, YT, XT, YTL, XTL; };
constexpr WgradSplitTile WGS_TILES[] = {
    {3, 128, 128, 4, 2, 3, 3}, {3, 64, 256, 4, 2, 1, 4}, {3, 32, 256, 2, 2, 1, 4},
    {1, 128, 384, 7, 4, 0, 0}, {1, 128, 256, 7, 4, 3, 6}, {1, 128, 128, 7, 4, 4, 4},
    {1, 64, 768, 4, 6, 0, 0},  {1, 64, 512, 4, 6, 0, 0},  {1, 64, 256, 4, 4, 2, 6}};
constexpr int WGS_N_TILES = 9;
// tiles of one plane that have an instantiation for images whose offsets fit 31 bits one by one only
constexpr bool wgb_far(int shape) { return shape == WGB_128x128 || shape == WGB_64x256; }
// LDS per buffer of dzdy; one plane: and a place for the octets that a thread does not have
inline int wgs_dzdy_bytes(const WgradSplitTile &t, int PYW) { return t.planes == 1 ? (t.TK * PYW + 1) * 16 : t.TK * PYW * 48; }
constexpr int WGB_MAX_HF = 5;      // filter heights whose derivative takes operands rounded to bf16

struct WgradSplitPlan {
    int shape;
    int TK, TR;
    bool linear;
    bool far;                // one plane: images in 31 bits one by one (wgrad_bf16_kernel)
    int NCH;                 // channels of the slab
    WgradSplitParams P;
    size_t lds_bytes;
    size_t partial_floats;   // 2 slots of TK*TR per block
    double us;               // estimated microseconds of the call
};

// Slab pitches in 32-bit words: lane r of an operand read is at word phase*PHP + fj*COLP + c*CHP + (row of the phase), and
// 32 lanes should fall into 32 banks.  The pitches with the fewest collisions of at most `limit` words a plane, smallest first.  For the
// plan that a call will use and for no other: lane by lane, for every shape tried, the 512 pairs of pitches took 0.2 ms of host time, longer
// than many a call.  The lanes of a filter column keep their distances whatever the pitches: their banks are one mask, turned.
inline void wgs_pitches(int NCH, int limit, WgradSplitParams *P) {
    struct Column { int col, chan; unsigned banks; };  // lanes of one column in different banks, from bank 0 on
    Column at[128];
    int first[5] = {}, groups = 0, n = 0;              // half-wave h: columns first[h] .. first[h + 1] - 1
    const int lanes = 32 * 4 < P->R ? 32 * 4 : (P->R + 31) / 32 * 32;
    for (int r = 0, ch = 0, fj = 0, fi = 0; r < lanes; ++r) {
        if (r % 32 == 0) first[groups++] = n;
        const unsigned bank = 1u << ((fi % P->Sh * P->PHP + fi / P->Sh) & 31);
        int a = first[groups - 1];
        while (a < n && (at[a].col != fj || at[a].chan != ch || (at[a].banks & bank))) ++a;
        if (a == n) at[n++] = Column{fj, ch, 0};
        at[a].banks |= bank;
        if (++fi == P->Hf) { fi = 0; if (++fj == P->Wf) { fj = 0; ++ch; } }
    }
    first[groups] = n;
    const int b0 = P->COLP, c0 = P->CHP - P->NP * P->RC * b0;
    long best = -1;
    WgradSplitParams B = *P;
    for (int b = 0; b < 16; ++b)
        for (int c = 0; c < 32; ++c) {
            const int colp = b0 + b, chp = P->NP * P->RC * colp + c0 + c;
            if (NCH * chp > limit || (best >= 0 && chp >= best)) break;
            // reads beyond the first, over the fullest bank of each half-wave; from `enough` on they cost more than the best pair so far
            int extra = 0;
            const int enough = best < 0 ? 128 : (int)((best - chp) * lanes / (4096 * 32)) + 1;
            for (int h = 0; h < groups && extra < enough; ++h) {
                unsigned bit[6] = {};                  // reads of each bank, as binary digits
                for (int a = first[h]; a < first[h + 1]; ++a) {
                    const unsigned turn = (unsigned)(at[a].col * colp + at[a].chan * chp) & 31;
                    unsigned carry = at[a].banks << turn | at[a].banks >> (-turn & 31);
                    for (int d = 0; carry; ++d) { const unsigned both = bit[d] & carry; bit[d] ^= carry; carry = both; }
                }
                unsigned fullest = ~0u;
                int most = 0;
                for (int d = 5; d >= 0; --d)
                    if (fullest & bit[d]) { fullest &= bit[d]; most |= 1 << d; }
                extra += most - 1;
            }
            const long cost = (long)extra * 4096 * 32 / lanes + chp;
            if (best < 0 || cost < best) { best = cost; B.COLP = colp; B.MPP = P->RC * colp; B.CHP = chp; }
        }
    *P = B;
}

// max(a, b, c), rounded where two of them are close, and a part of what the largest one hides
inline double overlapped(double a, double b, double c, double part) {
    const double most = a > b ? (a > c ? a : c) : (b > c ? b : c);
    const double x = a * a, y = b * b, z = c * c;
    return sqrt(sqrt(x * x + y * y + z * z)) + part * (a + b + c - most);
}

// One plane (wgrad_bf16_kernel): estimated microseconds of a call beyond its launches, and the schedule of kern_wgrad.h for it (nchunks = 0: equal
// ranges) on how many blocks: every block writes a piece of a tile that the fix-up pass has to read, so calls of few units take fewer
// blocks.  yt, xt: octets of the instantiation; first: passes over a sweep's first columns, per unit; lines: memory lines of 128 bytes per
// unit; filled: of a tile.  The constants are a fit to 63000 timed calls of 2170 random layers (several tiles, patches and schedules of
// each; off by 13 %, 1 standard deviation), but for the 4 us of the fix-up pass (1.65 in calls that follow one another slowly).
inline double wgb_us(const WgradSplitTile &tile, int NO, int yt, int xt, double first, double lines, int64_t tiles, int64_t NU, int n_cu, bool streams, double filled,
                     int *nchunks, int *nblocks) {
    constexpr double STEP[3] = {0.0561, 0.1165, 0.172}, FEWER[4] = {1.0, 0.583, 0.34, 0.198};        // by blocks of coefficients a wave; n_cu / 1, 2, 4, 8
    const double mfma = NO / 2 * STEP[tile.TK * tile.TR / 16384 - 1], stage = 0.0477 * yt + 0.05 * xt + 0.198 * first;
    const int64_t total = tiles * NU;
    double best = 1e300;
    for (int chunked = 0; chunked < 2; ++chunked)
        for (int f = 0; f < 4 && (f == 0 || total < 32 * n_cu); ++f) {
            const int nb = n_cu >> f;
            const int64_t nch = nb / tiles < NU ? nb / tiles : NU, blocks = chunked ? nch * tiles : total < nb ? total : nb;
            if (blocks < 1) continue;
            const double fetch = lines * (chunked ? (streams ? 2.59e-4 : 1.146e-4) : (streams ? 5.82e-4 : 2.61e-4)) * FEWER[f];
            const double pieces = blocks > 1 && !(chunked && nch == 1) ? 4.0 + 1.552e-6 * filled * (double)blocks * tile.TK * tile.TR : 0.0;
            const double us = overlapped(mfma, stage, fetch, 2.48) * (double)(chunked ? (NU + nch - 1) / nch : (total + blocks - 1) / blocks) + pieces;
            if (us < best) { best = us; *nchunks = chunked ? (int)nch : 0; *nblocks = nb; }
        }
    return best;
}

inline bool plan_wgrad_split_shape(const ConvView &v, int n_cu, int shape, bool streams, WgradSplitPlan *pl) {
    const WgradSplitTile tile = WGS_TILES[shape];
    const int TK = tile.TK, TR = tile.TR;
    const int T = v.Hf * v.Wf;
    const int64_t R64 = (int64_t)T * v.Cg;
    if (R64 >= ((int64_t)1 << 30)) return false;
    const int R = (int)R64, RT = (R + TR - 1) / TR, KT = (v.Kg + TK - 1) / TK;
    int NCH = 0;
    for (int rt = 0; rt < RT && rt <= T; ++rt) {       // the pattern repeats after T tiles
        const int lo = rt * TR, hi = lo + TR < R ? lo + TR : R, n = (hi - 1) / T - lo / T + 1;
        if (n > NCH) NCH = n;
    }
    const int64_t tiles = (int64_t)v.G * KT * RT;
    if (tiles >= ((int64_t)1 << 20)) return false;
    const int NPH = v.Hf < v.Sh ? v.Hf : v.Sh, XL = tile.planes == 1 ? (v.Pt + 3) / 4 * 4 : v.Pt;
    const int threads = 64 * WGS_STAGE_WAVES;
    // octets of x limited by rows of dzdy, columns by x itself: no output row may lie past the last row of x (one plane: rows of x past its last
    // one meet rows of dzdy that are zeroed)
    const bool linear = T == 1 && v.Sh == 1 && v.Sw == 1 && v.Pt == 0 && v.Pl == 0 && (tile.planes == 1 ? v.Ho <= v.H : v.Ho == v.H);
    // octets per staging thread of the instantiations there are (launch_wgrad_split)
    const int most_y = linear ? tile.YTL : tile.YT, most_x = linear ? tile.XTL : tile.XT;
    if (!most_y) return false;
    double best = 1e300;
    WgradSplitParams B = {};
    for (int TIQ = 1; TIQ <= 32; ++TIQ) {
        const int RB = (v.Ho + 4 * TIQ - 1) / (4 * TIQ);
        // fewer rows give the same row blocks; one plane: a second quad of rows that there are not, where nothing else makes the octets even
        if (TIQ > 1 && (v.Ho + 4 * TIQ - 5) / (4 * TIQ - 4) == RB && !(tile.planes == 1 && TIQ == 2 && v.Ho <= 4 && best >= 1e300)) continue;
        for (int NP = 1; NP <= 4; NP *= 2)
            for (int MC = 1; MC <= v.Wo && TIQ * MC * NP <= 32; ++MC) {
                const int NO = TIQ * MC * NP;
                if (NO & 1) continue;
                // one plane: a second pair of images that there is not, where nothing else makes the octets even
                if (NP > 1 && NP > (v.N + 1) / 2 && !(tile.planes == 1 && NP == 2 && MC == 1 && best >= 1e300)) continue;
                int TI = (v.Ho + RB - 1) / RB < 4 * TIQ ? (v.Ho + RB - 1) / RB : 4 * TIQ;      // rows shared out evenly
                const int YW = TK * NO;
                if (YW > most_y * threads) break;
                const int SC = (MC - 1) * v.Sw + v.Wf;
                // by 16-byte loads rows of x above the patch's first one come as whole quads, none of which may begin above the plane and reach into it:
                // where a second patch still reaches above it, patches are whole quads too
                if (tile.planes == 1 && RB > 1 && TI < XL) TI = 4 * TIQ;
                const int XQ = (4 * TIQ - 1 + (v.Hf - 1 + XL - v.Pt) / v.Sh) / 4 + 1;        // quads of a phase
                const int64_t XW1 = (int64_t)NCH * NP * NPH * XQ;
                const int step = MC * v.Sw < SC ? MC * v.Sw : SC, RC = 2 * SC;
                if (tile.planes == 1 && (step > 255 || 4 * XQ > 4095)) break;              // the staging waves keep a word's place in 32 bits
                if (XW1 * step > most_x * threads || (tile.planes == 3 && XW1 * (SC - step) > 2 * threads)) break;
                const int PHP = 4 * XQ, COLP = NPH * PHP, MPP = RC * COLP, CHP = NP * MPP;
                const int PYW = NO | 1, XPL = NCH * (CHP + NP * RC * 4 + 8);         // room for pitches: wgs_pitches
                const size_t lds = 2 * (size_t)wgs_dzdy_bytes(tile, PYW) + (size_t)XPL * 4 * tile.planes + 16;
                if (lds > IGEMM_LDS_LIMIT) break;
                const int CC = (v.Wo + MC - 1) / MC, IB = (v.N + 2 * NP - 1) / (2 * NP);
                bool far = false;
                if (tile.planes == 1) {
                    // bytes of a unit's images in 31 bits, with the columns that a sweep moves over; else one pair, an image in 31 bits and such a move in 30
                    const double xcol = 4.0 * v.H, ycol = 4.0 * v.Ho, ximage = xcol * v.W * v.Ctot, yimage = ycol * v.Wo * v.Ktot, moves = (double)CC * MC * v.Sw + v.Pl + SC;
                    far = 2 * NP * ximage + xcol * moves >= 2147483647.0 || 2 * NP * yimage >= 2147483647.0;
                    if (far && (NP > 1 || !wgb_far(shape) || ximage >= 2147483647.0 || yimage >= 2147483647.0 || xcol * (moves + 1) + ycol >= 1073741824.0 ||
                                ycol * ((double)CC * MC + 2) >= 1073741824.0 || xcol * ((double)v.W * NCH + v.Pl) >= 2147483647.0)) break;
                }
                // Microseconds of a unit: its MFMAs, splitting what it stages, fetching that (memory lines of 128 bytes), and of the
                // whole call.
                const int64_t NU = (int64_t)RB * CC * IB, total = tiles * NU;
                const int kn = v.Kg < TK ? v.Kg : TK, images = 2 * NP < v.N ? 2 * NP : v.N;
                const double extra = (double)(SC - step) / CC, columns = step + extra;
                const double lines = (double)kn * images * (TI == v.Ho ? MC * TI / 32.0 + 1.0 : MC * (TI / 32.0 + 1.0)) +
                                     (double)NCH * images * columns * (((TI - 1) * v.Sh + v.Hf) / 32.0 + 1.0);
                int nchunks = 0, nblocks = n_cu;
                double us;
                if (tile.planes == 1) {
                    const int rows = TI + v.Hf - 1 < v.H ? TI + v.Hf - 1 : v.H;                     // of x
                    const int xt = linear || XW1 * step > most_x / 2 * threads ? most_x : most_x / 2;      // of the instantiation
                    // dzdy in one run of whole columns, x likewise
                    const double run_lines = (double)kn * images * (TI == v.Ho ? MC * TI / 32.0 + 1.0 : MC * (TI / 32.0 + 1.0)) +
                                             (double)NCH * images * (RB == 1 ? columns * rows / 32.0 + 1.0 + extra : columns * (rows / 32.0 + 1.0));
                    const double first = (double)((XW1 * (SC - step) + 2 * threads - 1) / (2 * threads)) / CC;
                    us = wgb_us(tile, NO, most_y, xt, first, run_lines, tiles, NU, n_cu, streams, (v.Kg < TK ? (double)v.Kg / TK : 1.0) * (R < TR ? (double)R / TR : 1.0), &nchunks, &nblocks);
                } else {
                    // The constants are a fit to 31000 timed calls of 13400 random layers (several tiles and patches of each; the estimate is off by
                    // 8 %, 1 standard deviation).
                    const double mfma = NO / 2 * (TK == 32 ? 0.245 : 0.47);
                    const double split = 0.865 + 0.228 * ((YW + threads - 1) / threads) + (linear ? 0.222 : 0.308) * (double)((XW1 * step + threads - 1) / threads) +
                                         0.67 * XW1 * extra / threads;
                    const double unit = overlapped(mfma, split, lines * (streams ? 1.84e-3 : 1.09e-3), 0.225);
                    us = unit * (double)((total + n_cu - 1) / n_cu);
                    // The two schedules of kern_wgrad.h; chunks for arrays that stream from memory, at most one to a compute unit, if they are
                    // estimated to be faster or keep the compute units about as busy (they read the arrays fewer times).
                    if (streams && tiles <= n_cu) {
                        const int64_t nch = n_cu / tiles < NU ? n_cu / tiles : NU;
                        const double chunked = overlapped(mfma, split, lines * 1.48e-3, 0.225) * (double)((NU + nch - 1) / nch);
                        if (chunked < us || (double)total >= 0.95 * n_cu * (double)((NU + nch - 1) / nch)) { us = chunked; nchunks = (int)nch; }
                    }
                }
                if (us < best) {
                    best = us;
                    pl->far = far;
                    B.TI = TI; B.RB = RB; B.MC = MC; B.CC = CC; B.SC = SC; B.NP = NP; B.IB = IB; B.TIQ = TIQ; B.NO = NO; B.PYW = PYW; B.nchunks = nchunks; B.nblocks = nblocks;
                    B.NPH = NPH; B.XQ = XQ; B.PHP = PHP; B.COLP = COLP; B.MPP = MPP; B.CHP = CHP; B.YW = YW; B.XW1 = (int)XW1; B.XL = XL; B.RC = RC; B.step = step;
                }
            }
    }
    if (best >= 1e300) return false;
    WgradSplitParams &P = pl->P;
    P = B;
    P.H = v.H; P.W = v.W; P.N = v.N; P.Ctot = v.Ctot; P.Cg = v.Cg;
    P.Ho = v.Ho; P.Wo = v.Wo; P.Ktot = v.Ktot; P.Kg = v.Kg; P.G = v.G;
    P.Hf = v.Hf; P.Wf = v.Wf; P.Sh = v.Sh; P.Sw = v.Sw; P.Pt = v.Pt; P.Pl = v.Pl;
    P.xsj = v.H; P.xsc = v.H * v.W; P.xsn = v.H * v.W * v.Ctot; P.xtot = (long long)P.xsn * v.N;
    P.ysj = v.Ho; P.ysc = v.Ho * v.Wo; P.ysn = v.Ho * v.Wo * v.Ktot; P.ytot = (long long)P.ysn * v.N;
    // 32-bit byte offsets inside a unit's images
    if (tile.planes == 3 && ((double)v.H * v.W * v.Ctot * 8 * P.NP >= 2147483647.0 || (double)v.Ho * v.Wo * v.Ktot * 8 * P.NP >= 2147483647.0)) return false;
    P.KT = KT; P.RT = RT; P.R = R; P.tiles = (int)tiles;
    const int64_t NU = (int64_t)P.RB * P.CC * P.IB;
    if (NU >= ((int64_t)1 << 30)) return false;
    P.NU = (int)NU;
    P.dRB = make_div32(P.RB); P.dCC = make_div32(P.CC);
    P.dXW1 = make_div32(P.XW1); P.dXQ = make_div32(P.XQ); P.dNPH = make_div32(P.NPH); P.dNP = make_div32(P.NP);
    const int64_t total = tiles * NU;
    P.nblocks = P.nchunks > 0 ? (int)tiles * P.nchunks : (int)(total < P.nblocks ? total : P.nblocks);
    P.walk = make_sk_walk(P.nchunks > 0 ? NU : total, P.nchunks > 0 ? P.nchunks : P.nblocks, P.NU);
    pl->shape = shape; pl->TK = TK; pl->TR = TR;
    pl->linear = linear;
    pl->NCH = NCH;
    pl->partial_floats = P.nblocks > 1 && P.nchunks != 1 ? (size_t)2 * P.nblocks * TK * TR : 0;
    const double filled = (v.Kg < TK ? (double)v.Kg / TK : 1.0) * (R < TR ? (double)R / TR : 1.0);        // of a tile
    pl->us = tile.planes == 1 ? best : 12.7 + best + (pl->partial_floats ? 0.298 * 8e-6 * filled * P.nblocks * TK * TR : 0.0);
    return true;
}

// Estimated microseconds of a call on the fp32 kernel, from the same calls: off by 14 %.
inline double wgrad_fp32_us(const ConvView &v, const WgradPlan &pl, int n_cu) {
    const WgradParams &P = pl.P;
    const int lanes = pl.wino ? pl.TR / 3 : pl.TR, R = pl.wino ? v.Wf * v.Cg : P.R;
    const double rate = pl.shape == WG_64x192 ? 1.2023 : pl.shape == WG_32x256 ? 1.0474 : pl.shape == WG_96x128 ? 0.9502 : pl.shape == WG_96x384 ? 1.2412 : 1.1706;
    const double resident = P.nblocks > n_cu && pl.occupancy > 1 ? 2.0 : 1.0, rounds = ceil((double)P.nblocks / (n_cu * pl.occupancy));
    const int kn = v.Kg < pl.TK ? v.Kg : pl.TK, SRC = P.SRP * P.SC;
    const double lines = (double)kn * P.MC * (P.TI / 32.0 + 1.0) + (double)P.XS / SRC * (SRC / 32.0 + P.MC);
    const double mfma = pl.TK * lanes / 1024 / 4.0 * P.PCH / 2 * 64.0 / 2400.0 * rate * resident, fetch = 1.631 + resident * lines * 1.3143e-3;
    const double unit = overlapped(mfma, fetch, 0.0, 0.421);
    const double filled = (v.Kg < pl.TK ? (double)v.Kg / pl.TK : 1.0) * (R < lanes ? (double)R / lanes : 1.0);
    return 13.1 + rounds * ceil((double)P.tiles * P.NU / P.nblocks) * unit + 0.2884 * 4e-6 * (double)pl.partial_floats * filled;
}

// The filter derivative of `view` on the three-plane kernel; fp32: its plan on the fp32 kernel, or NULL if there is none.  False where the
// fp32 kernel is the faster one.  Over 15600 other random layers: always fp32 1.437 s, by this rule 1.031 s, the faster of the two each time
// 1.019 s; of the 10687 that it sends to three planes 87 are slower there by more than 2 %, 44 by more than 5 %.  The 4 us: calls of 15 to
// 20 us are launches, and the estimates do not tell their kernels apart.
inline bool plan_wgrad_split(const ConvView &view, int n_cu, const WgradPlan *fp32, WgradSplitPlan *pl, int planes = 3) {
    ConvView v = view;
    if (v.Hf == 1 && v.Wf == 1 && v.Sh == 1 && v.Sw == 1 && v.Pt == 0 && v.Pl == 0 && v.H == v.Ho && v.W == v.Wo) {
        v.H = v.Ho = v.H * v.W;          // a plane is one column
        v.W = v.Wo = 1;
    }
    const bool streams = 4.0 * ((double)v.H * v.W * v.Ctot + (double)v.Ho * v.Wo * v.Ktot) * v.N > 64.0 * 1024 * 1024;
    bool ok = false;
    for (int shape = 0; shape < WGS_N_TILES; ++shape) {
        const int TK = WGS_TILES[shape].TK;
        if (WGS_TILES[shape].planes != planes || (TK == 32 ? v.Kg > 32 : v.Kg <= TK / 2)) continue;
        WgradSplitPlan one;
        if (plan_wgrad_split_shape(v, n_cu, shape, streams, &one) && (!ok || one.us < pl->us)) { *pl = one; ok = true; }
    }
    if (!ok || (fp32 && pl->us >= wgrad_fp32_us(view, *fp32, n_cu) - 4.0)) return false;
    WgradSplitParams &P = pl->P;
    const int dzdy = 2 * wgs_dzdy_bytes(WGS_TILES[pl->shape], P.PYW);
    wgs_pitches(pl->NCH, ((int)IGEMM_LDS_LIMIT - dzdy - 16) / (4 * planes), &P);
    P.XPL = pl->NCH * P.CHP;
    P.counts = dzdy + planes * P.XPL * 4;
    pl->lds_bytes = (size_t)P.counts + 16;
    return true;
}

// Fully-connected forward (fc_forward_view): a lane's octet takes rows of a pair of images and there is one image only, so the R terms of a
// result go as two images of R/2.  Odd R: false.  6x6x256 -> 4096, 256 images: 233 us on the fp32 kernel, 198 here; of 49 layers of 1x1 to
// 7x7 inputs, 128 to 4096 channels, 16 to 256 images, 500 to 4096 filters the rule of plan_wgrad_split sends 29 here, which are 1.12 to 1.58 times
// as fast (median 1.35), with half of the error against 64 bits; none is slower.
inline bool plan_fc_forward_split(const Geom &g, int n_cu, const WgradPlan *fp32, WgradSplitPlan *pl) {
    ConvView v = fc_forward_view(g);
    const int R = v.H;
    if (R % 2) return false;
    v.H = v.Ho = R / 2; v.N = 2;
    if (!plan_wgrad_split(v, n_cu, fp32, pl)) return false;
    WgradSplitParams &P = pl->P;
    P.xsn = P.ysn = R / 2; P.xsc = P.ysc = R;          // offsets inside a unit stay below those that plan_wgrad_split has checked
    return true;
}

// ---- small layers (kern_small.h) ----------------------------------------------------------
// Which layers go there, by the products of a pass and the results it has.  Measured on 300 layers of 1 to 8 images of 8 to 53 samples a side, 3 to 32 channels,
// 4 to 64 filters of 1 to 5 taps a side, strides 1 to 3: forward up to 9e6 products 13.9 -> 9.3 us a call in the mean, none slower by more than 3 %, dzdx 20.4 -> 13.2,
// 10 slower, by 14 % at most; from there to 5e7 forward 18.9 -> 12.3, dzdx 33 -> 11, where more results than 4096 a channel leave the tiles of the
// other kernels enough to do.
// 1x1 filters gain nothing (14x9x24, eight filters, three images 12.2 -> 13.0).
inline bool small_sum(const Geom &g, int64_t pixels) {
    if (g.Hf * g.Wf == 1) return false;
    const double products = (double)g.Ho * g.Wo * g.N * g.K * g.Hf * g.Wf * g.Df;
    return products <= 9e6 || (products <= 5e7 && pixels <= 4096);
}

struct SmallPlan {
    SmallParams P;
    int views, blocks;       // stride phases, blocks of 64 pixels of the largest
    size_t lds_bytes;
};
// the next view of a plan
inline bool add_small_view(const ConvView &v, SmallPlan *pl) {
    SmallParams &P = pl->P;
    if (pl->views == SMALL_VIEWS) return false;
    if (pl->views == 0) {
        P.H = v.H; P.W = v.W; P.Ctot = v.Ctot; P.Cg = v.Cg; P.OH = v.OH; P.OW = v.OW; P.Ktot = v.Ktot; P.Kg = v.Kg;
        P.KT = (v.Kg + SMALL_K - 1) / SMALL_K;
        P.dKT = make_div32(P.KT);
        const int64_t bytes = (int64_t)v.H * v.W * v.Ctot * v.N * 4;
        if (bytes >= ((int64_t)1 << 30) || (int64_t)v.G * P.KT > 65535) return false;
        P.in_bytes = (int)bytes;
        pl->lds_bytes = sizeof(float) * SMALL_WAVES * SMALL_K * 64;
    }
    SmallView &S = P.v[pl->views++];
    const PlainView V = plain_view(v, false);
    S.Ho = v.Ho; S.Wo = v.Wo; S.pixels = v.Ho * v.Wo * v.N; S.Hf = v.Hf; S.Wf = v.Wf; S.Sh = v.Sh; S.Sw = v.Sw; S.Pt = v.Pt; S.Pl = v.Pl;
    S.oi0 = v.oi0; S.osi = v.osi; S.oj0 = v.oj0; S.osj = v.osj;
    S.wo = V.wo; S.wg = V.wg; S.wk = V.wk; S.wc = V.wc; S.wi = V.wi; S.wj = V.wj;
    S.dHo = make_div32(v.Ho); S.dWo = make_div32(v.Wo); S.dT = make_div32(v.Hf * v.Wf); S.dHf = make_div32(v.Hf);
    pl->blocks = std::max(pl->blocks, (S.pixels + 63) / 64);
    const size_t weights = sizeof(float) * (size_t)v.Cg * v.Hf * v.Wf * SMALL_K;
    pl->lds_bytes = std::max(pl->lds_bytes, weights);
    return weights <= (size_t)SMALL_LDS;
}

struct SmallFilterPlan {
    SmallFilterParams P;
    int grid;                // blocks of dzdw
};
inline bool plan_small_filter(const Geom &g, SmallFilterPlan *pl) {
    SmallFilterParams &P = pl->P;
    const int64_t xb = numel_x(g) * 4, yb = numel_y(g) * 4;
    if (g.Hf > SMALL_HF || xb >= ((int64_t)1 << 30) || yb >= ((int64_t)1 << 30)) return false;
    P.pieces = (g.Ho * g.Wo + BIAS_PIECE - 1) / BIAS_PIECE; P.dPieces = make_div32(P.pieces);
    P.H = g.H; P.W = g.W; P.D = g.D; P.N = g.N; P.Df = g.Df; P.K = g.K; P.Kg = g.Kg; P.KT = (g.Kg + SMALL_K - 1) / SMALL_K;
    P.Hf = g.Hf; P.Wf = g.Wf; P.Sh = g.Sh; P.Sw = g.Sw; P.Pt = g.Pt; P.Pl = g.Pl; P.Ho = g.Ho; P.Wo = g.Wo; P.pixels = g.Ho * g.Wo * g.N;
    P.x_bytes = (int)xb; P.y_bytes = (int)yb;
    P.dHo = make_div32(g.Ho); P.dWo = make_div32(g.Wo); P.dWf = make_div32(g.Wf); P.dDf = make_div32(g.Df); P.dKT = make_div32(P.KT);
    P.blocks = pl->grid = g.G * P.KT * g.Df * g.Wf;
    // A thread's pixels follow one another, each as long as its loads, and every block reads the whole of its filters' dzdy: 400 layers, up to 1024 pixels and 512
    // blocks 12.1 -> 9.2 us a call, up to 4096 and 256 13.2 -> 11.0; beyond, 15 -> 22.
    return P.pixels <= 256 * SMALL_PIXELS ? P.blocks <= 512 : P.pixels <= 4096 && P.blocks <= 256;
}

}  // namespace mcn
