// SkWalk against the plain divisions, and the fix-up passes' rule for a tile's pieces (sk_has_piece over all ranks) against sk_tile_pieces.
#include <stdio.h>
#include <stdlib.h>
#include "streamk.h"
using namespace mcn;

int main() {
    unsigned long long seed = 88172645463325252ull;
    auto rnd = [&](int lo, int hi) { seed ^= seed << 13; seed ^= seed >> 7; seed ^= seed << 17; return lo + (int)(seed % (unsigned long long)(hi - lo + 1)); };
    static int want[2048], got[2048];
    for (int c = 0; c < 20000; ++c) {
        const int nblocks = c % 3 ? 8 * rnd(1, 64) : rnd(1, 512), nshare = nblocks % 16 == 0 && c % 2 ? nblocks / 2 : nblocks;
        const int NU = c % 5 ? rnd(1, 400) : rnd(1, 1 << 29), tiles = rnd(1, c % 7 ? 60 : 2000);
        const long long total = (long long)tiles * NU;
        const SkWalk w = make_sk_walk(total, nshare, NU);
        for (int r = 0; r <= nshare; ++r) {
            const long long b = sk_begin(w, r);
            if (b != sk_begin(total, nshare, r) || (b < total && sk_tile(w, b, NU) != (int)(b / NU))) { printf("range %d of %d: %lld units, %d\n", r, nshare, total, NU); return 1; }
        }
        for (int k = 0; k < 4; ++k) {
            const int ts = rnd(0, tiles - 1);
            const long long lo = (long long)ts * NU, hi = lo + NU;
            const int n = sk_tile_pieces(total, NU, nblocks, nshare, ts, want, 2048);
            int m = 0;
            bool alone = false;
            for (int r = 0; r < nshare; ++r) {
                const long long bb = sk_begin(w, r), be = sk_begin(w, r + 1);
                if (!sk_has_piece(bb, be, lo, hi)) continue;
                alone |= bb <= lo && be >= hi;
                got[m++] = 2 * sk_share_block(nblocks, nshare, r) + (bb >= lo ? 0 : 1);
            }
            if (alone) m = 0;
            bool same = m == n;
            for (int i = 0; i < m && same; ++i) same = got[i] == want[i];
            if (!same) { printf("tile %d of %d: %d units, %d of %d blocks\n", ts, tiles, NU, nshare, nblocks); return 1; }
        }
    }
    printf("OK\n");
    return 0;
}
