// SkWalk against the plain divisions, the fix-up passes' rule for a tile's pieces (sk_has_piece over all ranks) against sk_tile_pieces, and the
// words that their blocks share (sk_dealt_word).
#include <stdio.h>
#include <stdlib.h>
#include <algorithm>
#include <vector>
#include "streamk.h"
using namespace mcn;

// Every word of a tile of `rows` filters, `groups` of 16 words each, once; at most `most` of the groups at one place of all filters in one block.
static bool dealt(int rows, int groups, int blocks, int per_pass, int most) {
    const int n = 16 * rows * groups;
    std::vector<int> taken(n, 0), load(groups * blocks, 0);
    for (int pass = 0; pass * blocks * per_pass * 16 < n; ++pass)
        for (int b = 0; b < blocks; ++b)
            for (int q = 0; q < 16 * per_pass; ++q) {
                const int w = sk_dealt_word(pass * per_pass + (q >> 4), blocks, make_div32(blocks), b, q & 15);
                if (w < 0) return false;
                if (w >= n) continue;
                ++taken[w];
                if (q % 16 == 0) ++load[w / 16 % groups * blocks + b];
            }
    return std::count(taken.begin(), taken.end(), 1) == n && *std::max_element(load.begin(), load.end()) <= most;
}

int main() {
    for (int rows : {1, 5, 32, 64, 100, 128})
        for (int groups : {1, 2, 3, 4, 6, 8, 12})
            for (int per_pass : {1, 2, 4, 8, 16})
                for (int blocks = 1; blocks <= 1024; blocks += blocks < 40 ? 1 : 61)
                    if (!dealt(rows, groups, blocks, per_pass, rows)) { printf("%d rows of %d groups, %d blocks, %d a pass\n", rows, groups, blocks, per_pass); return 1; }
    // one place of all filters of the tiles that there are, over a power of two of blocks: three times its even share at most (from the same block every round: all of them in one)
    for (int rows : {32, 64, 128})
        for (int groups : {2, 4, 6, 8, 12})
            for (int blocks = 2; blocks <= 256; blocks *= 2)
                if (!dealt(rows, groups, blocks, 16, 3 * ((rows + blocks - 1) / blocks))) { printf("%d rows of %d groups in few of %d blocks\n", rows, groups, blocks); return 1; }
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
