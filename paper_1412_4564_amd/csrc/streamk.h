// The stream-K split of the left-over tiles (kern_igemm.h, kern_wgrad.h): which block computes which units, and
// which pieces a shared tile consists of.  Plain integer arithmetic; the header also compiles as C++ on the host,
// where tests/streamk_check.cpp and streamk_walk_check.cpp compare the pieces with a simulation of the blocks' walk over their ranges.
#pragma once
#include "fastdiv.h"

namespace mcn {

// Blocks on consecutive hardware ids land on different XCDs; give each XCD a contiguous
// share of the work so that neighbouring tiles (shared halo, same weights) meet in one L2.
MCN_HOST_DEVICE inline int sk_virtual_block(int b, int nblocks) {
    return (nblocks % 8 == 0) ? (b % 8) * (nblocks / 8) + b / 8 : b;
}
// Block vb of nblocks (at most 46340) holds the units [total*vb/nblocks, total*(vb+1)/nblocks).  With total = q * nblocks + r,
// total * vb / nblocks = q * vb + r * vb / nblocks; q and r are found on the host: a 64-bit division is some 150 scalar instructions
// one after another, and a block that does four of them before its first load starts 2 us later.
struct SkWalk {
    long long q;
    unsigned r;
    Div32 n, NU;                    // r * vb < n^2 < 2^31
};
inline SkWalk make_sk_walk(long long total, int nblocks, int NU) {
    return SkWalk{total / nblocks, (unsigned)(total % nblocks), make_div32(nblocks), make_div32(NU)};
}
MCN_HOST_DEVICE inline long long sk_begin(const SkWalk &w, int vb) { return w.q * vb + div32((int)(w.r * (unsigned)vb), w.n); }
MCN_HOST_DEVICE inline int sk_tile(const SkWalk &w, long long unit, int NU) { return unit <= 0x7fffffff ? div32((int)unit, w.NU) : (int)(unit / NU); }

// Rank of virtual block vb among the nshare sharing blocks (in virtual order), or -1; and its inverse.  With
// nshare < nblocks (both multiples of 8) the sharing blocks are hardware ids 0 .. nshare-1, i.e. the first
// nshare/8 virtual blocks of each XCD's run of nblocks/8.
MCN_HOST_DEVICE inline int sk_share_rank(int nblocks, int nshare, int vb) {
    if (nshare == nblocks) return vb;
    const int G = nblocks / 8, S = nshare / 8;
    const int x = vb / G, i = vb - x * G;
    return i < S ? x * S + i : -1;
}
MCN_HOST_DEVICE inline int sk_share_block(int nblocks, int nshare, int r) {
    if (nshare == nblocks) return r;
    const int G = nblocks / 8, S = nshare / 8;
    return (r / S) * G + r % S;
}

// The pieces of a tile (units [t_lo, t_hi)) as the fix-up passes find them, from the ranges [bb, be) of the blocks: whether a block holds one;
// whether it holds a certain unit (kern_wgrad.h: the first and the last one's blocks, all between them hold a piece); and where the
// piece is: a block's first segment is its slot 0, any later one that is not a whole tile its slot 1.  A block that holds all of a tile
// stores the tile itself.
MCN_HOST_DEVICE inline bool sk_has_piece(long long bb, long long be, long long t_lo, long long t_hi) { return be > bb && be > t_lo && bb < t_hi; }
MCN_HOST_DEVICE inline bool sk_holds(long long bb, long long be, long long unit) { return bb <= unit && unit < be; }
MCN_HOST_DEVICE inline int sk_slot(int block, long long bb, long long t_lo) { return 2 * block + (bb >= t_lo ? 0 : 1); }

// The 16-byte words of a tile as the blocks of a fix-up pass that forms sums again share them: in groups of 16, one a round for each of the
// tile's `blocks`, round j from j blocks further back than the one before.  A filter's groups then lie in several blocks, also where a round
// ends among them, and so do those of one place in all filters, whatever the distance between them (every round from the next block on,
// that distance and `blocks` could leave them to a few; groups at a round's end and the next one's beginning went to one block).
MCN_HOST_DEVICE inline int sk_dealt_word(int round, int blocks, Div32 dBlocks, int block, int in_group) {
    const int back = round * (round + 1) / 2, turned = block - (back - div32(back, dBlocks) * blocks);
    return 16 * (round * blocks + (turned < 0 ? turned + blocks : turned)) + in_group;
}

// Dealt unit order of a tile cut into nchunks chunks, one per block (kern_wgrad.h, WgradParams::deal).  Chunk c
// holds the q or q + 1 units [NU*c/nchunks, NU*(c+1)/nchunks) by count; the chunks c0 .. c0 + n - 1 of the blocks on
// one XCD cover one contiguous range between them, and their blocks take its units in turn: in round k < q block i
// takes unit base + n*k + i, and in the last, partial round the blocks with q + 1 units take the rest in block order.
struct DealSplit {
    int n, q, i, base, n_long;      // chunks on the XCD, units per short chunk, this chunk's place among them,
                                    // first unit of the XCD's range, chunks before this one with q + 1 units
};
MCN_HOST_DEVICE inline DealSplit make_deal(int NU, int nchunks, int n, int chunk) {
    DealSplit d;
    const int q = NU / nchunks, rem = NU - q * nchunks;          // rem * chunk < nchunks^2: 32 bits for nchunks <= 32768
    const int c0 = (chunk / n) * n;
    d.n = n; d.q = q; d.i = chunk - c0;
    d.base = q * c0 + rem * c0 / nchunks;
    d.n_long = rem * chunk / nchunks - rem * c0 / nchunks;
    return d;
}
MCN_HOST_DEVICE inline int dealt_unit(const DealSplit &d, int k) { return d.base + d.n * k + (k < d.q ? d.i : d.n_long); }

}  // namespace mcn
