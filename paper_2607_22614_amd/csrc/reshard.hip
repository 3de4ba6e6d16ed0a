// Reshard kernel: the training -> training move to a new shard count
// (weights and optimizer states from the old training ranks to the new ones).
// The N elements keep their order and bits; they are re-cut into W' shards and
// the destination padding is zeroed.  Same tiling and checksum scheme as the
// stage kernel, with one fp32 word per element: a lane moves a
// 16-byte group (one nontemporal load, one nontemporal store).  HBM-bound: 4 B
// read and 4 B written per element (padding: written only).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "device_common.h"
#include "kernels.h"

namespace dr {
namespace {

struct ReshardArgs {
  const DevSeg* segs;
  const Tile* tiles;
  ChunkSum sum;              // the chunks' checksum accumulators and output slots
  uint64_t chunk_elems;      // B / 4
  uint64_t dst_shard_elems;  // S'
  uint32_t tile0, ntiles;
  uint32_t part_shift;       // log2 of the parts that a workgroup each moves of a tile (reshard_kernel)
  float* flat;               // non-null: write destination element e to flat[e - flat_bias] (one chunk)
  uint64_t flat_bias;
  const float* src[DR_MAX_SHARDS];
  float* dst[DR_MAX_SHARDS];
};

// K groups per lane of tile g, from the tile's unit `first` on: loads, stores and adds the
// checksum sums.  Every lane of the workgroup calls it.
template <int K>
__device__ __forceinline__ void reshard_tile(const ReshardArgs& a, uint32_t g, uint32_t first,
                                             uint64_t (*red)[kThreads / 64]) {
  const Tile tile = load_tile(a.tiles, g);
  const DevSeg s = load_seg(a.segs, tile.seg);
  const uint32_t unit0 = tile.unit0 + first;
  if (unit0 >= s.units) return;
  float* __restrict__ out = a.flat ? a.flat + (s.dst - a.flat_bias)
                                   : a.dst[s.dst_shard] + (s.dst - (uint64_t)s.dst_shard * a.dst_shard_elems);
  const uint64_t pos0 = s.dst - (uint64_t)s.chunk * a.chunk_elems;  // word position in the chunk
  const uint32_t last = s.units - 1;
  uint64_t acc_w = 0, acc_rw = 0;
  if (s.op == DR_OP_ZERO_F32) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t u = unit0 + k * kThreads + threadIdx.x;
      if (u <= last) store_stream((f32x4){0.f, 0.f, 0.f, 0.f}, reinterpret_cast<f32x4*>(out + 4 * u));
    }
  } else {
    const float* __restrict__ src = a.src[s.shard] + s.src;
    u32x4 v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t u = min(unit0 + k * kThreads + threadIdx.x, last);
      v[k] = load_stream(reinterpret_cast<const u32x4*>(src + 4 * u));
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t u = unit0 + k * kThreads + threadIdx.x;
      if (u <= last) {
        store_stream(v[k], reinterpret_cast<u32x4*>(out + 4 * u));
        const uint32_t e = 4 * u;  // word index relative to the segment
        acc_w += (uint64_t)v[k].x + v[k].y + (uint64_t)v[k].z + v[k].w;
        acc_rw += (uint64_t)e * v[k].x + (uint64_t)(e + 1) * v[k].y + (uint64_t)(e + 2) * v[k].z +
                  (uint64_t)(e + 3) * v[k].w;
      }
    }
  }
  block_sum2(acc_w, acc_rw, red);
  if (threadIdx.x == 0) add_tile_sums(a.sum, g, s.chunk, acc_w, (pos0 + 1) * acc_w + acc_rw);
}

// kHalves: a workgroup moves half a tile, two 16-byte groups per lane, and the XCDs take groups of 32
// halves (256 KiB) in turn; else it moves a whole tile and each XCD streams through one eighth.
// Bound by HBM, where the read and the write stream meet in the same banks: how they fall together
// depends on the tile's size, on the order and on where the buffers lie.  Mean over five placements
// of the buffers (24, 32 and 44 layers 8 to 6: fourteen) with their standard deviation, in us, whole /
// halves, back to back; after 30 ms idle:
//   0.5B, 8 to 6 shards (5.0 GB)  825+-18 / 790+-3; 861 / 825      odd width, 5 to 3 (5.4)  943+-4 / 877+-15; 975 / 910
//   8B width, 8 layers, 4 to 16 (22.3)  3651+-16 / 3560+-47; 3678 / 3605
//   16 layers, 8 to 6 (36.3)  5811+-158 / 5650+-55; 5894 / 5816    20 (43.3)  6882+-230 / 6764+-29; 6931 / 6849
//   24 layers (50.3)  7793+-73 / 7860+-48; 7839 / 7963             28 (57.2)  8817+-118 / 8946+-30; 8902 / 9056
//   32 layers (64.2)  9962+-328 / 10045+-64; 10008 / 10142         32, 8 to 3  10094 / 10076; 10186 / 10200
//   32, 4 to 16  10036 / 10029; 10076 / 10145                      44 (85)  13248+-70 / 13358+-86; 13285 / 13497
//   32B width, 20 layers (91)  14130 / 14185; 14177 / 14350
// So halves up to kWholeTileBytes, whole tiles beyond (launch_reshard).  Halves in groups of 16 / 64 /
// 128 instead of 32 at 16 layers: 5882 / 5700 / 5655, at 32 layers 10602 / 10169 / 10180; halves in
// contiguous order 5763 and 9931 back to back, but 5993 and 10190 after idle; whole tiles in groups
// or in plain order 5868-6189 and 10489-11055.
template <bool kHalves>
__global__ __launch_bounds__(kThreads) void reshard_kernel(ReshardArgs args) {
  (void)args;  // read through the kernarg segment (same bytes)
  const ReshardArgs& a = *(const ReshardArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  __shared__ uint64_t red[2][kThreads / 64];
  if (!kHalves) {
    for (uint32_t b = blockIdx.x; b < a.ntiles; b += gridDim.x)
      reshard_tile<kReshardIters>(a, a.tile0 + xcd_tile(b, a.ntiles), 0, red);
    return;
  }
  const uint64_t n = (uint64_t)a.ntiles << a.part_shift;
  for (uint64_t b = blockIdx.x; b < n; b += gridDim.x) {
    const uint64_t t = xcd_group<kPartGroup>(b, n);
    const uint32_t part = (uint32_t)t & ((1u << a.part_shift) - 1);
    reshard_tile<kPartIters>(a, a.tile0 + (uint32_t)(t >> a.part_shift), part * kPartIters * kThreads, red);
  }
}

// The path through host memory: packs tiles [tile0, tile0 + ntiles) into pinned host memory (flat)
// and reloads what the previous launch packed into the destination shards, in alternation
// (the reason is at the stage kernel's form).  A step is half a tile, 8 KiB each way.  2.7 GB each
// way in 8 MiB chunks, 5 to 3 shards: 77.5 -> 60.4 ms (a packing kernel and copies before).
struct ReshardRelayArgs {
  ReshardArgs s;
  const u32x4* from;  // pinned, 16-byte groups of the previous launch
  uint64_t elem0;     // destination element of the first group
  uint32_t groups;
  uint32_t shard0;    // destination shard of elem0
};

__global__ __launch_bounds__(kThreads) void reshard_relay_kernel(ReshardRelayArgs args) {
  (void)args;  // read through the kernarg segment (same bytes)
  const ReshardRelayArgs& a = *(const ReshardRelayArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  __shared__ uint64_t red[2][kThreads / 64];
  constexpr uint32_t per = kThreads * kPartIters;
  const uint32_t reloads = (a.groups + per - 1) / per, packs = a.s.ntiles * kTileParts, steps = max(packs, reloads);
  const uint64_t S2 = a.s.dst_shard_elems;
  for (uint32_t b = blockIdx.x; b < steps; b += gridDim.x) {
    const uint32_t u0 = b * per + threadIdx.x;
    u32x4 v[kPartIters];
    if (b < reloads) {
#pragma unroll
      for (int k = 0; k < kPartIters; ++k) v[k] = load_stream(a.from + min(u0 + k * kThreads, a.groups - 1));
    }
    if (b < packs) reshard_tile<kPartIters>(a.s, a.s.tile0 + b / kTileParts, b % kTileParts * per, red);
    if (b < reloads) {
#pragma unroll
      for (int k = 0; k < kPartIters; ++k) {
        const uint32_t u = u0 + k * kThreads;
        if (u < a.groups) {
          const uint64_t e = a.elem0 + 4ull * u;
          uint32_t w = a.shard0;  // at most DR_MAX_SHARDS - 1 steps: e lies in the destination
          while (e >= (uint64_t)(w + 1) * S2) ++w;
          store_stream(v[k], reinterpret_cast<u32x4*>(a.s.dst[w] + (e - (uint64_t)w * S2)));
        }
      }
    }
  }
}

}  // namespace

namespace {

ReshardArgs reshard_args(const ReshardLaunch& l) {
  ReshardArgs args;
  std::memset(&args, 0, sizeof(args));
  args.segs = l.segs;
  args.tiles = l.tiles;
  args.sum = l.sum;
  args.chunk_elems = l.chunk_elems;
  args.dst_shard_elems = l.dst_shard_elems;
  args.tile0 = l.tile0;
  args.ntiles = l.ntiles;
  args.flat = l.flat;
  args.flat_bias = l.flat_bias;
  for (int w = 0; w < l.num_src; ++w) args.src[w] = l.src[w];
  if (l.dst)
    for (int w = 0; w < l.num_dst; ++w) args.dst[w] = l.dst[w];
  return args;
}

}  // namespace

hipError_t launch_reshard_kernel(const ReshardLaunch& l, hipStream_t st) {
  if (!l.ntiles) return hipSuccess;
  ReshardArgs args = reshard_args(l);
  if (l.whole_tiles) {
    hipLaunchKernelGGL(reshard_kernel<false>, dim3(std::min(l.ntiles, kMaxGrid)), dim3(kThreads), 0, st, args);
    return hipGetLastError();
  }
  args.part_shift = reshard_part_shift(l.chunk_elems);
  const uint64_t grid = std::min<uint64_t>((uint64_t)l.ntiles << args.part_shift, kMaxGrid);
  hipLaunchKernelGGL(reshard_kernel<true>, dim3((uint32_t)grid), dim3(kThreads), 0, st, args);
  return hipGetLastError();
}

hipError_t launch_reshard_relay(const ReshardLaunch& l, const Reload& r, hipStream_t st) {
  if (!l.ntiles && !r.groups) return hipSuccess;
  ReshardRelayArgs args;
  args.s = reshard_args(l);
  args.from = static_cast<const u32x4*>(r.from);
  args.elem0 = r.elem0;
  args.groups = r.groups;
  args.shard0 = (uint32_t)(r.elem0 / l.dst_shard_elems);
  constexpr uint32_t per = kThreads * kPartIters;
  const uint32_t steps = std::max(l.ntiles * kTileParts, (r.groups + per - 1) / per);
  hipLaunchKernelGGL(reshard_relay_kernel, dim3(std::min(steps, kReshardRelayGrid)), dim3(kThreads), 0, st, args);
  return hipGetLastError();
}

}  // namespace dr
