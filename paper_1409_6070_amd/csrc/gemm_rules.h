// Rules of the gather GEMMs that the device code and the launch code share.  constexpr,
// so a host program can run the same text.
#pragma once

#include <stdint.h>

namespace sscn {

constexpr int XCDS = 8;  // workgroups go round-robin to the eight XCDs, each with its own L2

// Several column tiles to a gathered row tile: consecutive workgroups take tiles
// ntiles / 8 apart, so that a row tile's column tiles and its neighbours read their
// rows through one L2.  (DeepCNet(5,50) at batch 1600: 145.6 -> 137.1 us for the third
// forward, 225.2 -> 217.9 for the third input gradient; at batch 100 13.9 -> 13.2 and
// 19.2 -> 18.9.  One column tile, or the softmax layer's few rows, lose by it: 16.2 ->
// 16.9, 29.3 -> 48.9.)
constexpr inline bool deal_by_xcd(int tiles_n, bool gathered, int A, int ksplit) {
  return tiles_n > 1 && gathered && A > 1 && ksplit == 1;
}

// Workgroups of a launch of up to `tiles` tiles: one a tile, at most `limit` (a
// multiple of XCDS), and dealt by XCD the same number on each, so that none of them
// takes a tile more than in plain order.  (With the odd workgroups on the first XCDs
// only, a launch whose tiles filled its grid ran two tiles on some: 64 x 64 tiles of
// a DeepCNiN(4,43) at batch 419, 315 on a grid of 315, 22.0 -> 14.9 us for a forward
// and 18.7 -> 13.2 for an input gradient; 924 on 924 of a float32 DeepCNet(2,99) at
// batch 461, 46.9 -> 35.6.)
constexpr inline int deal_grid(int64_t tiles, int limit, bool by_xcd) {
  int64_t g = tiles < 1 ? 1 : tiles < limit ? tiles : limit;
  if (by_xcd) g = (g + XCDS - 1) / XCDS * XCDS;
  return (int)g;
}

// The tiles first, first + step, .. < end of workgroup `block` of `grid`.
struct TileDeal {
  int first, end, step;
};
constexpr inline TileDeal deal_tiles(int ntiles, int grid, int block, bool by_xcd) {
  if (!by_xcd) return TileDeal{block, ntiles, grid};
  const int xcd = block % XCDS, per = (ntiles + XCDS - 1) / XCDS;
  const int end = (xcd + 1) * per;
  return TileDeal{xcd * per + block / XCDS, end < ntiles ? end : ntiles, (grid + XCDS - 1 - xcd) / XCDS};
}

// Kernel instantiations (template value) by what the epilogue does: plain, the
// pooling forward, the masked store EPI_STORE_MASK; 0 or 4 the pooling backward with
// that window count.
constexpr int PLAIN_MODE = -1, POOL_FWD_MODE = -2, MASK_MODE = -3;

// The instantiation of a launch.  Split K writes partial sums, and the reduce behind
// it masks them: that is a plain launch (the masked one loads the tile of the layer
// below before its K loop, for every K range: DeepCNiN(5,50) at batch 100, the input
// gradient above the topmost 1x1 layer below the last, K in five ranges, float32 16.9
// us against 15.8 with its reduce).
constexpr inline int gemm_mode(bool pool_fwd, bool masked, bool route, int route_ac, int ksplit) {
  if (pool_fwd) return POOL_FWD_MODE;
  if (masked && ksplit == 1) return MASK_MODE;
  return route ? (route_ac == 4 ? 4 : 0) : PLAIN_MODE;
}

}  // namespace sscn
