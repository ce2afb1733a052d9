// schedule.h -- the shapes and orders of the stage launches, host code without
// a device call: work-groups of the LDS-staged variants, column orders of large
// boxes.
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
// planes (us, 12-real, FP32 full, FP64): 32x32x96x96 1982, 2891, 6669 against
// 1913, 2695, 6434 / 1850, 2626, 6331 / 1867, 2656, 6298; 16x16x48x48 x 6 (192
// tiles per slice) 700, 892, 1775 against, for 4 / 8 / 16 planes, 687, 843,
// 1668 / 690, 849, 1687 / 697, 873, 1734.
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

}  // namespace tgf
