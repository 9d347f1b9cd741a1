// Which tiles the workgroups of a register-resident kernel take.  Plain C++ for both sides: the kernels run it on the GPU, the tests run
// the same functions on the CPU.
#pragma once

#include "draw.hpp"

namespace quasar {

// floor(T * b / G) for wave-uniform non-negative operands: where a workgroup's share of T tiles
// begins.  The 64-bit division is a long software routine; it runs only when the product does
// not fit 32 bits.
QUASAR_BOTH int tile_split(int T, int b, int G) {
    const unsigned long long prod = (unsigned long long)(unsigned int)T * (unsigned int)b;
    if (prod <= 0xFFFFFFFFull) return (int)((unsigned int)prod / (unsigned int)G);
    return (int)(prod / (unsigned long long)(unsigned int)G);
}

// Contiguous shares without a division: of G workgroups each has q tiles and the FIRST r one more (q = T / G, r = T % G), where
// tile_split spreads those over all of them.  The two are not interchangeable: what reads by the cuts of tile_split (the sampler's
// blocks, sample.hpp) needs them, and a vocabulary of 151936 takes 108 us cut like this and 99.9 like that.
QUASAR_BOTH int share_begin(int q, int r, int b) { return b * q + (b < r ? b : r); }
QUASAR_BOTH int share_count(int q, int r, int b) { return q + (b < r ? 1 : 0); }

// The tiles of workgroup b, in units of TU: p.tq of them and one more in the first p.tr workgroups, which lie alike in the XCDs of a slice.
// DEAL: round by round, unit u in the u-th stretch of p.groups units, the workgroups of an XCD side by side in it, so that the chip
// walks the matrix from front to back and an XCD reads a megabyte or two at a time (without regard to the XCDs 16384 x 8192, M = 32
// is 29.1 us, so 27.3, contiguous 28.2).  Else contiguous: EVEN as tile_split cuts, or
// share_begin.
template <int TU, bool DEAL, bool EVEN>
struct TileShare {
    static constexpr bool kDeal = DEAL;
    int first, step, rest, units, tq;   // unit u < tq begins at tile first + u * step, unit tq at tile `rest`; units in all
    template <class P>
    QUASAR_BOTH TileShare(const P &p, int b) : tq(p.tq) {
        units = share_count(p.tq, p.tr, b);
        if constexpr (DEAL) {
            // behind the workgroups of the XCDs in front of its own, which have groups >> shift or one more
            const int mask = (1 << p.xcd_shift) - 1;
            first = TU * (share_begin(p.groups >> p.xcd_shift, p.groups & mask, b & mask) + (b >> p.xcd_shift));
            step = TU * p.groups;
            rest = tq * step + TU * b;
        } else if constexpr (EVEN) {
            first = TU * tile_split(p.T / TU, b, p.groups);
            units = tile_split(p.T / TU, b + 1, p.groups) - first / TU;
        } else {
            first = TU * share_begin(p.tq, p.tr, b);
        }
    }
    QUASAR_BOTH int tile(int tl) const {
        if constexpr (!DEAL) return first + tl;
        const int u = TU == 2 ? tl >> 1 : tl;
        return (u < tq ? first + u * step : rest) + (TU == 2 ? tl & 1 : 0);
    }
};

// p.T tiles in units of TU over `groups` workgroups of each of `ksplit` slices of K
template <class P>
inline void share_tiles(P &p, int groups, int ksplit, int TU) {
    p.groups = groups;
    p.tq = p.T / TU / groups;
    p.tr = p.T / TU % groups;
    // Workgroup b of slice s is the launch's (s + ksplit * b)th, and workgroup i of a launch lies in XCD i mod 8: those of a slice lie by turns
    // in 8 XCDs, 4 (two or six slices), 2 (four) or 1 (eight).  us, int8, shares of three, five, six and seven slices dealt without regard to
    // that, so: 16384 x 14336 M = 12 42.4, 41.4, 8192 x 25600 M = 32 42.5, 41.8, 16384 x 17408 M = 24 56.2, 54.3, 5120 x 14336 M = 24 18.0,
    // 18.0 (contiguous 42.2, 42.2, 56.1, 18.0).
    const int common = ksplit & -ksplit;     // the power of two in it
    p.xcd_shift = common >= 8 ? 0 : (common == 4 ? 1 : (common == 2 ? 2 : 3));
}

}  // namespace quasar
