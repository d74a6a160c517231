// rbf_split.h -- what the pairwise kernel's launch and the ranges that a weight gradient's
// points are split into must agree on: the LDS tile and the hinges per block.
#pragma once

#include <cstdint>

#include "pdmp_common.h"

namespace pdmp {

// Chunks of one LDS tile of the pairwise kernel: whole rows of 16 chunks, rounded up from 64
// KiB (2-D: 1,376 chunks, 512 bytes more), so that no hinge set or range of points that fits
// 64 KiB is split: a second tile is restaged in every step (5,456 hinges: 114 us against 55
// for 4 steps of 5,000 samples).
template <int DIM>
constexpr int rbf_tile_chunks() { return (tile_chunks<DIM>() + 15) / 16 * 16; }

// Lanes are hinges there: two per lane halve the LDS reads that bind it, unless the last
// block of 512 then idles for more than an eighth of the work (40,001 points, 3-D, 1,044
// hinges: 1,536 lanes' work in three such blocks, 1,280 in five of 256).
inline int wgrad_hinges_per_block(int64_t M) {
    const int64_t two = (M + 511) / 512 * 512, one = (M + 255) / 256 * 256;
    return 8 * two <= 9 * one ? 512 : 256;
}

}  // namespace pdmp
