// The ranges of units and the pieces of a tile, found by divisions and one block after another: what the rules of csrc/streamk.h, by which the
// kernels find them, are checked against.
#pragma once
#include "streamk.h"

namespace mcn {

inline long long sk_begin(long long total, int nblocks, int vb) { return total * vb / nblocks; }

// The pieces of left-over tile ts (units [ts*NU, (ts+1)*NU) of `total`), in the order in which they are added: workspace slots
// 2*block + segment.  The sharing block of rank r holds the units [total*r/nshare, total*(r+1)/nshare); the first rank with units of
// this tile follows from one division (and a step of correction); its piece is its first segment if its range starts in this tile, else
// its second; the pieces of the following ranks are first segments.  Returns the number of pieces, 0 when one block computed the whole
// tile (it stored the tile itself), at most max_pieces.
inline int sk_tile_pieces(long long total, int NU, int nblocks, int nshare, int ts, int *slots, int max_pieces) {
    const long long t_lo = (long long)ts * NU, t_hi = t_lo + NU;
    int first = (int)(t_lo * nshare / total);
    while (first + 1 < nshare && sk_begin(total, nshare, first + 1) <= t_lo) ++first;
    while (first > 0 && sk_begin(total, nshare, first) > t_lo) --first;
    int n = 0;
    for (int b = first; b < nshare && n < max_pieces; ++b) {
        const long long bb = sk_begin(total, nshare, b);
        if (bb >= t_hi) break;
        const long long be = sk_begin(total, nshare, b + 1);
        if (be == bb || be <= t_lo) continue;                        // a block without units of this tile wrote nothing
        if (bb <= t_lo && be >= t_hi) return 0;                      // one block computed the whole tile
        slots[n++] = 2 * sk_share_block(nblocks, nshare, b) + (bb >= t_lo ? 0 : 1);
    }
    return n;
}

}  // namespace mcn
