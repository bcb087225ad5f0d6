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

// Site chunks of the weight gradients.  A network with few tiles plans chunks of a
// half or a quarter (div 2 or 4) of the standard length; how long a pass makes them
// is decided from the tiles that its own rows give at each length (convolutions of
// both tile widths together): the shortest of a quarter with at most 512 tiles, a half
// with at most 700, and the standard length.  Below that a launch leaves compute units
// idle and a chunk is a serial loop; above, shorter chunks only multiply the partial
// sums.  Weight gradients and their reduce, in us at the standard length / a half / a
// quarter, with the tiles: DeepCNet(4,20), float32, batch 8 (32 / 57 / 108 tiles) 45.7 /
// 36.1 / 25.8; from paths, bf16, batch 100 (83 / 158 / 310) 36.0 / 28.1 / 28.2;
// DeepCNet(5,64), batch 7 (147 / 210 / 338) 36.1 / 27.7 / 26.3; DeepCNet(4,77), batch 16
// (259 / 388 / 686) 35.3 / 28.7 / 32.1; DeepCNiN(4,40), batch 100 (362 / 691 / 1346)
// 42.3 / 36.9 / 45.8; DeepCNet(3,50), batch 300 (322 / 630 / 1237) 39.9 / 40.6 / 51.4;
// DeepCNet(4,100), batch 30 (428 / 769 / 1416) 38.6 / 40.3 / 46.5; DeepCNiN(2,60), batch
// 1500 (384 / 766 / 1273) 59.2 / 61.8 / 69.8.
// Returns the multiple (1 .. div) of the planned length; tiles[i]: at a multiple of 2^i.
constexpr inline int chunk_multiple(int div, int64_t const (&tiles)[3]) {
  if (div == 4 && tiles[0] <= 512) return 1;
  if (div >= 2 && tiles[div == 4 ? 1 : 0] <= 700) return div / 2;
  return div;
}

}  // namespace sscn
