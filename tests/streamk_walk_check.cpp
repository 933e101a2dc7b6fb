// SkWalk against the plain divisions, the fix-up passes' rules for a tile's pieces against sk_tile_pieces (igemm: sk_has_piece over all ranks;
// filter derivative: the blocks that hold its first and its last unit, sk_holds, and all between them), and the words that their blocks
// share (sk_dealt_word).
#include <stdio.h>
#include <stdlib.h>
#include <algorithm>
#include <vector>
#include "streamk_reference.h"
using namespace mcn;

// Every word of a tile of `rows` filters, C4 words each, once; at most `most` of those of one channel's 25 coefficients (seven words of each
// filter) in one block; and the groups of a filter each in another, where there are more blocks than rounds.
static bool dealt(int rows, int C4, int blocks, int per_pass, int most) {
    const int n = rows * C4, rounds = (n + 16 * blocks - 1) / (16 * blocks), passes = (rounds + per_pass - 1) / per_pass;
    std::vector<int> block_of(n, -1), load(blocks), seen(blocks, -1);
    for (int pass = 0; pass < passes; ++pass)
        for (int b = 0; b < blocks; ++b)
            for (int q = 0; q < 16 * per_pass; ++q) {
                const int w = sk_dealt_word(pass * per_pass + (q >> 4), blocks, make_div32(blocks), b, q & 15);
                if (w < 0 || (w < n && block_of[w] >= 0)) return false;
                if (w < n) block_of[w] = b;
            }
    if (std::count(block_of.begin(), block_of.end(), -1)) return false;
    for (int c = 0; c < C4; c += 7) {
        std::fill(load.begin(), load.end(), 0);
        for (int k = 0; k < rows; ++k)
            for (int w = c; w < c + 7 && w < C4; ++w) ++load[block_of[k * C4 + w]];
        if (*std::max_element(load.begin(), load.end()) > most) return false;
    }
    for (int k = 0; k < rows && blocks > rounds + C4 / 16 + 2; ++k)
        for (int g = k * C4 / 16; g <= (k * C4 + C4 - 1) / 16; ++g) {
            const int b = block_of[g * 16 < k * C4 ? k * C4 : g * 16];
            if (seen[b] == k) return false;
            seen[b] = k;
        }
    return true;
}

// The pieces of a tile as wgrad_fixup_kernel finds them: no block's range is empty (no more blocks than units), so one block holds the tile's first
// unit and one its last.
static bool ends(int tiles, int NU, int blocks) {
    const long long total = (long long)tiles * NU;
    const int n = blocks < total ? blocks : (int)total;
    const SkWalk w = make_sk_walk(total, n, NU);
    std::vector<int> want(n + 1);
    for (int i = 0; i < 4; ++i) {
        const int ts = i == 0 ? 0 : i == 1 ? tiles - 1 : (int)((unsigned)(i * 7919 * (tiles + n)) % (unsigned)tiles);
        const long long lo = (long long)ts * NU, hi = lo + NU;
        int found[3] = {-1, -1, -1}, hits = 0;
        for (int b = 0; b < n; ++b) {
            const long long bb = sk_begin(w, b), be = sk_begin(w, b + 1);
            if (bb >= be) { printf("block %d of %d is empty: %lld units\n", b, n, total); return false; }
            if (sk_holds(bb, be, lo)) { found[0] = b; found[2] = sk_slot(b, bb, lo); ++hits; }
            if (sk_holds(bb, be, hi - 1)) { found[1] = b; ++hits; }
        }
        const int pieces = found[1] - found[0] + 1, k = sk_tile_pieces(total, NU, n, n, ts, want.data(), n + 1);
        bool same = hits == 2 && (pieces < 2 ? k == 0 : pieces == k);
        for (int j = 0; j < k && same; ++j) same = want[j] == (j == 0 ? found[2] : 2 * (found[0] + j));
        if (!same) { printf("ends of tile %d of %d: %d units, %d blocks\n", ts, tiles, NU, n); return false; }
    }
    return true;
}

int main() {
    for (int tiles : {1, 2, 3, 7, 64})
        for (int NU : {1, 2, 3, 5, 16})
            for (int blocks : {1, 2, 3, 8, 64, 255, 256, 1024})
                if (!ends(tiles, NU, blocks)) return 1;
    for (int rows : {1, 5, 32, 64, 100, 128})
        for (int C4 : {1, 7, 12, 16, 32, 48, 64, 96, 128, 144, 192})
            for (int per_pass : {1, 2, 4, 8, 16})
                for (int blocks = 1; blocks <= 512; blocks += blocks < 40 ? 1 : 59)
                    if (!dealt(rows, C4, blocks, per_pass, 7 * rows)) { printf("%d rows of %d words, %d blocks, %d a pass\n", rows, C4, blocks, per_pass); return 1; }
    // a channel's words: four times a block's even share of them at most, to the next group (every round from the next block on: up to twelve times)
    for (int rows : {64, 128})
        for (int C4 : {12, 24, 32, 48, 64, 96, 128, 192})
            for (int blocks = 4; blocks <= 85 && 2 * blocks <= rows * C4 / 16; ++blocks)
                if (!dealt(rows, C4, blocks, 16, 4 * 7 * rows / blocks + 7)) { printf("a channel of %d rows of %d words in few of %d blocks\n", rows, C4, blocks); return 1; }
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
                got[m++] = sk_slot(sk_share_block(nblocks, nshare, r), bb, lo);
            }
            if (alone) m = 0;
            bool same = m == n;
            for (int i = 0; i < m && same; ++i) same = got[i] == want[i];
            if (!same) { printf("tile %d of %d: %d units, %d of %d blocks\n", ts, tiles, NU, nshare, nblocks); return 1; }
        }
        if (!ends(tiles, NU, nblocks)) return 1;
    }
    printf("OK\n");
    return 0;
}
