// Shapes of the row-flattened tiles (stencil_rf.hpp, stencil_les_rf.hpp) as
// functions of the grid's sizes alone.  Host code without HIP, so that a test
// can evaluate it anywhere.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "kl.h"

namespace kl {

// Row-flattened tiles: rows of cpr = ceil(itot / vx) chunks, R whole rows per
// block of at most `threads` threads.  A block also needs a thread for every
// chunk of its two halo rows, and LDS for RF_PLANES planes of R + 2 rows and a
// spare chunk per lane: blocks of 256 threads take rows of up to 80 chunks
// (three rows, 52 KB, three blocks on a CU), blocks of 512 up to 256 (two rows,
// 122 KB).
constexpr int RF_PLANES = 7;  // u: 2, v: 2, w: 3
inline int rf_chunks(int itot, int vx) { return (int)(((int64_t)itot + vx - 1) / vx); }
inline int rf_max_chunks(int threads) { return threads == 256 ? 80 : 256; }
inline int rf_rows(int jtot, int cpr, int threads)
{
    const int most = threads / cpr < jtot ? threads / cpr : jtot;
    const int blocks = (jtot + most - 1) / most;
    return (jtot + blocks - 1) / blocks;  // row blocks of equal height
}
inline size_t rf_lds_bytes(int cpr, int R) { return (size_t)RF_PLANES * ((R + 2) * cpr + 64) * 16; }
constexpr size_t RF_LDS_256 = (size_t)RF_PLANES * (5 * 80 + 64) * 16, RF_LDS_512 = (size_t)RF_PLANES * (4 * 256 + 64) * 16;

// Levels per tile in a launch of nby row blocks: about 512 tiles (two per CU),
// at least two levels each; longer marches read less twice, more tiles balance
// better, and no other power of two was faster by more than 3% at the sizes
// tried (64^3 .. 320x320x160, odd rows, both types).  A block of 512 threads has
// its CU to itself, so those tiles run in rounds of 256, and 300 of them leave
// the second round nearly empty.  Where a march that fills the chip (240 tiles; the
// fused pass at 384x380x64 FP32 took 63 us with 228, 57 with 456) needs a tenth
// less, a tile costing five levels more than it computes, that one is taken:
// 832x600x64 FP32 diff_uvw 304 -> 246 us, fused step 316 -> 233; 492x635x214 FP64
// 1121 -> 940 and 1032 -> 762; 384x380x380 FP64 825 -> 739 and 856 -> 688.
inline int rf_levels(int nby, int ktot, int threads)
{
    const int per = std::max(1, 512 / nby), kb0 = std::max(2, (ktot + per - 1) / per);
    if (threads != 512) return kb0;
    auto tiles = [&](int kb) { return (int64_t)nby * ((ktot + kb - 1) / kb); };
    auto cost = [&](int kb) { return (double)((tiles(kb) + 255) / 256) * (kb + 5); };
    int best = kb0;
    double least = 0.9 * cost(kb0);
    for (int n = 1; n <= 16 && 8 * n <= ktot; ++n) {
        const int kb = (ktot + n - 1) / n;
        if (tiles(kb) >= 240 && cost(kb) < least) {
            least = cost(kb);
            best = kb;
        }
    }
    return best;
}

// Row-flattened tiles of the paper's schemes (stencil_les_rf.hpp): rows cut into
// the fewest segments of at most 64 (advec_u_2i5; 60 of two points) or 48
// (diff_smag) chunks, W each, and R rows, so that the block's chunks, the
// chunks around it (one per thread) and the LDS fit a block of 512 threads.
struct LesRfShape {
    int W, R, threads;
    size_t lds;
};
// Segment width.  Where the rows divide into 32 chunks (512 bytes; padding of
// less than 1/32 counts as dividing) a segment's lines are its own, and that is
// fastest; 64 for advec_u_2i5 at V = 4 (512x512x128 FP32, us by width: 64 115,
// 32 120, 43 150, 48 142; diff_smag 32 237, 43 313, 48 274).  Other rows: the
// fewest segments whose taller halo still fits (301x203x151 FP32, 76 chunks:
// 38 38.7, 26 44.9, 64 57.3); for three and more of diff_smag their width is
// rounded up to a cache line (151 chunks: 40 148, 38 165, 51 does not fit).
inline LesRfShape les_rf_shape(int kernel, int itot, int jtot, int vx)
{
    const bool a5 = kernel == KL_KERNEL_ADVEC_U_2I5;
    const int cpr = rf_chunks(itot, vx), wmax = a5 ? (vx == 4 ? 64 : 60) : 48, hc = 4 / vx;
    int W = cpr;
    if (cpr > wmax) {
        const int nsx = (cpr + wmax - 1) / wmax;
        if ((cpr + 31) / 32 * 32 - cpr <= cpr / 32)
            W = wmax == 64 && cpr % 64 == 0 ? 64 : 32;
        else
            W = (cpr + nsx - 1) / nsx;
        if (!a5 && nsx > 2) W = (W + 7) / 8 * 8;
    }
    auto extra = [&](int R) { return a5 ? 6 * W + 2 * hc * (R + 6) + W + 2 * R + 1 : 8 * W + 8 * (R + 2); };
    auto lds = [&](int R) {  // a chunk is 16 bytes
        return a5 ? (size_t)2 * ((R + 6) * (W + 2 * hc) + (2 * R + 1) * (W + 1) + 64) * 16
                  : (size_t)3 * (4 * (R + 2) * (W + 2) + 64) * 16;
    };
    int R = std::min(jtot, 512 / W);
    while (R > 1 && (extra(R) > 512 || lds(R) > 160 * 1024)) --R;
    const int blocks = (jtot + R - 1) / R;
    R = (jtot + blocks - 1) / blocks;
    return {W, R, (std::max(R * W, extra(R)) + 63) / 64 * 64, lds(R)};
}

// Levels per tile of `slab` tiles per level slab: the fewest rounds of 256
// tiles (one block per CU) times levels, a tile costing about five levels
// more than it computes (its prologue and its end).  Where fewer than four tiles
// make a slab, 64 slabs do not fill the CUs: then also as many as do.
inline int les_rf_levels(int slab, int ktot)
{
    int best = ktot;
    double least = 1e300;
    auto consider = [&](int nbz) {
        const int kb = (ktot + nbz - 1) / nbz;
        const double cost = (double)(((int64_t)slab * nbz + 255) / 256) * (kb + 5);
        if (cost < least) {
            least = cost;
            best = kb;
        }
    };
    for (int nbz = 1; nbz <= 64 && (nbz == 1 || 2 * nbz <= ktot); ++nbz) consider(nbz);
    for (int r = 1; slab < 4 && r <= 4; ++r)
        if (256 * r / slab * 2 <= ktot) consider(256 * r / slab);
    return best;
}

}  // namespace kl
