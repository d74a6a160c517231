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

// The pairwise weight gradient: a.M points as weighted hinges in a.splits ranges, a.n hinges
// as the lanes' samples, 256 or 512 of them per block.
int32_t launch_rbf_wgrad(int dim, const RbfArgs &a, int hinges_per_block, hipStream_t st);

}  // namespace pdmp
