// Which tile, and which elements of it, each workgroup and lane of the tile kernels takes.  Plain
// index arithmetic on the host and on the device, so that the CPU tests run what the kernels run.
#pragma once

#include <hip/hip_runtime.h>

#include "dev_types.h"

namespace dr {

// Tile run by the b-th workgroup: XCD x = b % 8 takes tiles
// [x*per + min(x, rem), ...) in order, where per/rem split n tiles over 8
// XCDs.  A bijection on [0, n) for every n.
__host__ __device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t n) {
  const uint32_t per = n / kXcds, rem = n % kXcds, x = b % kXcds;
  return x * per + (x < rem ? x : rem) + b / kXcds;
}

// Item run by the b-th workgroup in grouped order: the XCDs take groups of G consecutive items in
// turn, so the chip works on one window of 8*G items; the last n % (8*G) items in plain order.  A
// bijection on [0, n) for every n; item b of a full window runs on XCD b % 8.
template <uint32_t G, typename T>
__host__ __device__ __forceinline__ T xcd_group(T b, T n) {
  static_assert((G & (G - 1)) == 0, "power of two");
  if (b >= (n & ~(T)(kXcds * G - 1))) return b;
  const T x = b % kXcds, i = b / kXcds;
  return (i / G * kXcds + x) * G + i % G;
}

constexpr uint32_t kTileGroup = 64;  // tiles of a group in grouped order (stage, moment sums)

// Reshard: a workgroup's part of a tile (groups per lane), the parts of a group in grouped order, and
// log2 of the parts of a tile: one where a chunk, and so a tile, holds no more groups than a part.
constexpr int kPartIters = 2;
constexpr uint32_t kPartGroup = 32;
constexpr uint32_t kTileParts = kReshardIters / kPartIters;
static_assert(kTileParts == 2, "a tile is two parts");
__host__ __device__ __forceinline__ uint32_t reshard_part_shift(uint64_t chunk_elems) {
  return chunk_elems / 4 <= (uint64_t)kPartIters * kThreads ? 0 : 1;
}

// q = e / cols, r = e % cols for e < 2^32, from magic = floor(2^32 / cols):
// the estimate is at most one below the quotient, so one correction suffices.
__host__ __device__ __forceinline__ uint32_t div_cols(uint32_t e, uint32_t cols, uint32_t magic, uint32_t* rem) {
  uint32_t q = (uint32_t)((uint64_t)e * magic >> 32);
  uint32_t r = e - q * cols;
  if (r >= cols) {
    q += 1;
    r -= cols;
  }
  *rem = r;
  return q;
}

// Source offset of element e of a segment, and its column.
__host__ __device__ __forceinline__ uint32_t elem_src(const DevSeg& s, uint32_t e, uint32_t* col) {
  uint32_t row = 0;
  *col = e;
  if (s.rows > 1) row = div_cols(e, s.cols, s.magic, col);
  return row * s.stride + *col;
}

// Unaligned tiles of the stage kernel move groups of 4 elements, laid on the destination's 8-byte grid:
// group g of the segment holds its elements [4g - lead, 4g - lead + 4), where lead is the
// segment's first element modulo 4, so the first and the last group can be partial and a row can
// end inside a group.  The first element of lane `lane`'s k-th group of the tile at unit0:
__host__ __device__ __forceinline__ int32_t group_elem(uint32_t unit0, int k, uint32_t lane, uint32_t lead) {
  return (int32_t)(unit0 + 4 * (k * kThreads + lane)) - (int32_t)lead;
}
// Whether the group from element e on lies in the segment (one 8-byte store), and whether 16-byte
// loads bring it: one from elem_src(e), and if its row ends inside it after `cut` elements, one from
// (stride - cols) further, which holds elements [cut, 4) in their places.  Both lie between the group's
// first and last source element (the row after the cut belongs to the segment).
__host__ __device__ __forceinline__ bool whole_group(const DevSeg& s, int32_t e) {
  return e >= 0 && (uint32_t)e + 4 <= s.units;
}
__host__ __device__ __forceinline__ bool wide_group(const DevSeg& s, int32_t e) { return whole_group(s, e) && s.cols >= 4; }
__host__ __device__ __forceinline__ uint32_t group_cut(const DevSeg& s, uint32_t col) {
  return s.cols - col < 4 ? s.cols - col : 4;
}
// The groups of a segment's last tile end `lead` elements before the tile's last unit: up to three
// more elements, one lane each.
__host__ __device__ __forceinline__ bool tail_elem(const DevSeg& s, uint32_t unit0, uint32_t lane, uint32_t lead,
                                                   uint32_t* e) {
  *e = unit0 + kScalarUnitsPerTile - lead + lane;
  return lane < lead && unit0 + kScalarUnitsPerTile >= s.units && *e < s.units;
}

}  // namespace dr
