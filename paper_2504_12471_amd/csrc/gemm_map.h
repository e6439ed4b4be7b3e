// What the matrix-core products share: how operands are declared to the buffer loads and in which order workgroups take tiles.
#pragma once

#include "d2ft_common.h"

namespace d2ft {

constexpr uint32_t kBufBytes = 0x80000000u;   // declared buffer size; operands are checked to be smaller
// Any offset >= kBufBytes reads as zero, under any scalar offset below kBufBytes: the bounds check compares the lane's
// offset with the size less the scalar one.
constexpr uint32_t kOutside = 0x80000000u;

// The chip has 8 XCDs with one L2 each and workgroup ids are dealt to them round-robin, so ids with the same value mod 8 are
// renumbered to a contiguous range of tiles; inside that range tiles are walked in groups of 8 tile rows so that
// the workgroups resident on one XCD share A and B slabs through its L2.
__device__ __forceinline__ int xcd_range(int pid, int total) {
    const int xcd = pid & 7, idx = pid >> 3;
    return xcd * (total >> 3) + min(xcd, total & 7) + idx;
}
__device__ __forceinline__ void tile_at(int index, int tiles_m, int tiles_n, int& tm, int& tn) {
    constexpr int GM = 8;
    const int group = index / (GM * tiles_n);
    const int first = group * GM;
    const int gsize = min(tiles_m - first, GM);
    const int in_group = index - group * GM * tiles_n;
    tm = first + in_group % gsize;
    tn = in_group / gsize;
}
__device__ __forceinline__ void tile_of_block(int pid, int total, int tiles_m, int tiles_n, int& tm, int& tn, int& split) {
    const int lid = xcd_range(pid, total), per_split = tiles_m * tiles_n;
    split = lid / per_split;
    tile_at(lid - split * per_split, tiles_m, tiles_n, tm, tn);
}

}  // namespace d2ft
