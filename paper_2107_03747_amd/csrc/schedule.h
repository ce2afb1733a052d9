// schedule.h -- the shapes and orders of the stage launches, host code without
// a device call: work-groups of the LDS-staged variants, column orders of large
// boxes, the default variant.
#pragma once

#include <algorithm>

#include "layout.h"

namespace tgf {

// Sites per work-group of the LDS-staged stage variants: whole (n0, n1) planes
// (so that every neighbour in directions 0 and 1 lies in the block) when at
// least two of them fill half of the 256 threads; otherwise 256.  For the
// L x L x 3L x 3L boxes: L = 6 -> 252, 8 -> 256, 10 -> 200, 12 -> 144.
inline int default_block(const int d[4]) {
    const int plane = d[0] * d[1];
    if (plane > kBlock) return kBlock;
    const int k = kBlock / plane;
    return k * plane >= kBlock / 2 ? k * plane : kBlock;
}

// Column width of the LDS-staged launch order (block_order): site order while
// an n3 slice spans at most kChunkSlice work-groups (its direction-3
// neighbours are then among the work-groups an XCD runs at a time), else the
// largest divisor of the slice's work-group count up to kChunk.  Stage launch
// on the 32x32x96x96 box (384 work-groups per slice) against site order, for
// columns of 8 / 16 / 32 work-groups: FP32 12-real - / -6.3% / -6.8%,
// FP32 full -8.2% / -11.5% / -9.3%, FP64 -7.3% / -8.3% / +6.9% (the wider the
// column, the more of the XCD's L2 the direction-3 neighbours need; FP64
// holds 144 KB per work-group).
constexpr int kChunk = 16;
constexpr int kChunkSlice = 64;
inline int block_chunk(const int d[4], int blk) {
    const long long s = (long long)d[0] * d[1] * d[2];
    if (s % blk) return 0;
    const long long slice = s / blk;
    if (slice <= kChunkSlice) return 0;
    for (int ch = kChunk; ch >= 4; ch--)
        if (slice % ch == 0) return ch;
    return 0;
}

// Column width of the quad variant's 64-site tiles (tile_order): site order
// while an n3 slice spans at most kTileSlice tiles (about what an XCD runs at a
// time), else four (n0, n1) planes, or the largest divisor of the slice's tile
// count below that.  Stage launch, site order against columns of 2 / 4 / 8
// planes (us, 12-real and FP32 full): 32x32x96x96 1982, 2891 against 1913, 2695 /
// 1850, 2626 / 1867, 2656; 16x16x48x48 x 6 (192 tiles per slice) 700, 892
// against, for 4 / 8 / 16 planes, 687, 843 / 690, 849 / 697, 873.  FP64, site
// order and four planes: 6864 and 6546, 1815 and 1717.
constexpr int kTileSlice = 128;
inline int tile_chunk(const int d[4]) {
    const long long s = (long long)d[0] * d[1] * d[2];
    if (s % 64) return 0;
    const long long slice = s / 64, planes = std::max(16LL, 4LL * d[0] * d[1] / 64);
    if (slice <= kTileSlice) return 0;
    for (long long ch = std::min(planes, slice); ch >= 8; ch--)
        if (slice % ch == 0) return (int)ch;
    return 0;
}

// Does the stage of a configuration run in the LDS-staged kernel by default,
// not in the quad kernel?  By its extents and the storage alone, so that its
// results are those of a run of its own whatever batch it is in.  The quad
// kernel forms fewer loops where its tiles are closed under a shift, and fills
// the chip sooner; the LDS-staged kernel, where its work-groups are nearly full
// (>= 192 sites) and deep (>= 6 rows), finds more neighbours in them, which
// decides once a box is large:
//   - whole-plane work-groups (>= 224 sites) of rows that 64 does not hold
//     whole: FP32 full from 2^19 sites, 12-real from 2^21;
//   - else the full storages from 7 2^20 sites, unless only the quad kernel has
//     a column order for the box.
// Stage launch, quad and LDS-staged (us): FP32 full 9x9x81x81 155 and 145,
// 9x9x162x162 642 and 567, 6x6x252x252 654 and 567, 9x9x324x324 2853 and 2165,
// 32x32x96x96 2600 and 2550, 40x40x120x120 7518 and 6608; FP64 9x9x324x324
// 6513 and 5217, 24x24x128x128 6976 and 6322, 32x32x96x96 6575 and 6360;
// 12-real 9x9x162x162 470 and 454, 6x6x504x504 1954 and 1771.  On the other
// side of the lines: FP32 full 9x9x57x57 81 and 86, 16x16x160x160 1639 and
// 1692, 64x64x48x48 2727 and 2935; FP64 9x9x162x162 1300 and 1555,
// 18x18x144x144 4445 and 5185, 36x36x108x108 10397 and 11074; 12-real
// 9x9x108x108 208 and 215, 32x32x96x96 1862 and 1900.  Batches of many small
// boxes of such rows stay with the quad kernel (FP32 full, 60 of L = 9: 962
// and 900; one: 22 and 28); tgf_autotune times the whole batch.
inline bool lds_by_default(const int d[4], bool f64, bool c12) {
    const long long V = 1LL * d[0] * d[1] * d[2] * d[3];
    const int plane = d[0] * d[1], blk = default_block(d);
    if (64 % plane == 0 || blk < 192 || blk < 6 * d[0]) return false;
    if (!f64 && plane <= blk && blk >= 224 && 64 % d[0] != 0)
        return V >= (c12 ? 1LL << 21 : 1LL << 19);
    return !c12 && V >= 7LL << 20 && (block_chunk(d, blk) || !tile_chunk(d));
}

}  // namespace tgf
