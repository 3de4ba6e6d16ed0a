// Stage kernel: pack + cast + per-chunk checksum of the rollout stream on
// gfx950 (CDNA4), and the chunk-sum kernel.  The launches behind
// dr_stage_chunk / dr_stage_all are driven from staging.cpp.
//
// The work is a gather of contiguous runs with a narrowing cast: every output
// element is read once as fp32 and written once as bf16, so the kernel is
// bound by HBM bandwidth (6 bytes of traffic per element) and never touches
// MFMA.  Design points:
//   * the planner cuts the stream into segments that never cross a shard or
//     chunk boundary, and each workgroup tile lies inside one segment, so a
//     tile finds its work with two uniform (scalar) loads, its tile record and
//     then its segment record, and every lane of a tile takes the same branch;
//   * on aligned segments a lane moves groups of 4 elements: one 16-byte
//     nontemporal load, two packed round-to-nearest-even converts (two bf16
//     per instruction), one 8-byte nontemporal store.  Lane l of a wave takes
//     group l, so one wave instruction covers 1 KiB of source and 512 B of
//     destination, contiguous within a row;
//   * every load of a lane is issued before the first convert (K = 2 or 4
//     independent 16-byte loads in flight per lane: the plan's tile depth);
//   * segments that are no whole groups (column slices of an odd width) move
//     groups of 4 elements too, on the destination's 8-byte grid with 16-byte
//     loads at 4-byte boundaries.  Bound: as the aligned path, plus the rows'
//     partial lines.  A 12-layer decoder with 1821-element down slices on 3
//     ranks (4.05 GB, 27 % of it unaligned) took 693 us with one element per
//     lane, 4-byte loads and 2-byte stores, and takes 650 us; with the elements
//     of a group that a row ends in loaded one by one it took 661 us, with 1 or
//     4 groups per lane instead of 2 679-690 us;
//   * XCD-aware tile order: the hardware hands workgroup b to XCD b % 8, and
//     the kernel maps it to a tile so that each XCD streams through one
//     contiguous eighth of the stream instead of every eighth tile (measured
//     faster on the 8B shape: 6.3 vs 6.0 TB/s), or, in launches of up to a few
//     GiB, so that the XCDs take groups of 64 tiles in turn
//     (StageLaunch::grouped);
//   * the chunk checksum is accumulated from the packed words while they are
//     in registers, reduced across the wavefront (DPP moves, no LDS) and the
//     workgroup (LDS), and added with two 64-bit atomic adds (nothing waits
//     for them) into one of the chunk's accumulator slots; a small kernel
//     behind the launch adds a chunk's slots.  In small launches each tile
//     waits for its adds and the last one of a chunk adds the slots, with no
//     kernel behind.  The sums are integer, so the bits do not depend on the
//     order of the adds, and there is no extra pass over the data.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "device_common.h"
#include "kernels.h"

namespace dr {
namespace {

// Everything a stage launch needs, passed as the kernel's only argument.  The
// kernel reads it through the kernarg segment pointer, so the shard table is
// indexed with one scalar load instead of being copied into registers.
struct StageArgs {
  const DevSeg* segs;
  const Tile* tiles;
  uint16_t* dst;          // points at stream element dst_bias
  ChunkSum sum;           // the chunks' checksum accumulators and output slots
  uint64_t dst_bias;
  uint64_t chunk_elems;   // B / 2
  uint32_t tile0, ntiles; // tiles [tile0, tile0 + ntiles)
  uint32_t grid;          // workgroups of the launch, at most ntiles
  uint32_t grouped;       // 1: XCDs take groups of tiles in turn, 0: a contiguous eighth each
  const float* shards[DR_MAX_SHARDS];
};

// The convert below is exact only in the default FP mode: fast-math may
// assume no NaN or infinity, and a flush-to-zero denormal mode would flush
// fp32 subnormals before rounding.  Fast-math is refused here; the denormal
// mode of every kernel is checked in the built assembly by the test suite.
#if defined(__FAST_MATH__) || __FINITE_MATH_ONLY__
#error "stage.hip needs the default FP mode: build without -ffast-math / -ffinite-math-only"
#endif

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two fp32 -> one word of two bf16 (x in the low half), rounded to nearest
// with ties to even by gfx950's packed convert (v_cvt_pk_bf16_f32).  In the
// default FP mode it keeps fp32 subnormals (no flush), rounds overflow to
// infinity and returns a NaN as its upper half with the quiet bit set: equal
// to the integer definition on all 2^32 inputs, checked on the device.
__device__ __forceinline__ uint32_t cvt_pk_bf16(float x, float y) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x, y}, bf16x2));
}

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kGroups = kScalarIters / 4;  // groups of 4 elements per lane in an unaligned tile
static_assert(kScalarIters % 4 == 0, "unaligned tiles are whole groups per lane");

// load_stream of 4 elements at a 4-byte boundary (a template argument would lose the alignment).
__device__ __forceinline__ f32x4 load_stream4u(const float* p) {
#if DR_NT_LOADS
  return __builtin_nontemporal_load(reinterpret_cast<const f32x4u*>(p));
#else
  return *reinterpret_cast<const f32x4u*>(p);
#endif
}

// A group of an unaligned segment on its way: element j comes from a if j < cut, else from b.
struct Group {
  f32x4 a, b;
  uint32_t cut;
};

// Loads elements [e, e+4) of an unaligned segment, 0 for those outside [0, units): with one or two
// 16-byte loads at 4-byte boundaries (wide_group), the segment's ends and rows shorter than a
// group element by element, so nothing outside the segment's span is read.
__device__ __forceinline__ void load_group(const float* __restrict__ src, const DevSeg& s, int32_t e, Group& g) {
  uint32_t col;
  const uint32_t so = elem_src(s, (uint32_t)max(e, 0), &col);
  g.a = g.b = (f32x4){0.f, 0.f, 0.f, 0.f};
  g.cut = 4;
  if (wide_group(s, e)) {
    const float* p = src + so;
    g.a = load_stream4u(p);
    g.cut = group_cut(s, col);
    if (g.cut < 4) g.b = load_stream4u(p + (s.stride - s.cols));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (e + j < 0 || (uint32_t)(e + j) >= s.units) continue;
      g.a[j] = load_stream(src + elem_src(s, (uint32_t)(e + j), &col));
    }
  }
}

// Tile g of the tiling: loads, converts, stores and adds its checksum sums; K groups of 4 elements
// per lane on aligned segments; kOwnSums: in a launch that sums its chunks itself.  Every lane of the
// workgroup calls it.
template <int K, bool kOwnSums>
__device__ __forceinline__ void stage_tile(const StageArgs& a, uint32_t g, uint64_t (*red)[kThreads / 64]) {
  const Tile tile = load_tile(a.tiles, g);
  const DevSeg s = load_seg(a.segs, tile.seg);
  const float* __restrict__ src = a.shards[s.shard] + s.src;
  uint16_t* __restrict__ out = a.dst + (s.dst - a.dst_bias);
  // Checksum of the tile: word j of the chunk counts (j+1)*w_j.  With jb the
  // chunk word index of the segment's first group of 4 elements, j = jb + rel
  // where rel < 2^31 is the word index relative to that group, so lanes sum
  // A = sum w and R = sum rel*w with 32x32->64 multiply-adds and the tile's
  // s2 = (jb+1)*A + R is formed once at the end.
  const uint64_t pos0 = s.dst - (uint64_t)s.chunk * a.chunk_elems;  // element position in the chunk
  const uint32_t lead = (uint32_t)(pos0 & 3);  // elements of the first group before the segment (0 if aligned)
  uint64_t acc_w = 0, acc_rw = 0;
  const uint32_t last = s.units - 1;

  if (__builtin_expect((s.flags & DR_SEG_VEC4) != 0, 1)) {
    const bool contiguous = s.rows == 1;
    f32x4 v[K];
    // Loads first, all unconditional: lanes past the end of a ragged tile
    // re-read the segment's last group and store nothing.
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t u = min(tile.unit0 + k * kThreads + threadIdx.x, last);
      const uint32_t e = u * 4;
      uint32_t so = e;
      if (!contiguous) {
        uint32_t col;
        const uint32_t row = div_cols(e, s.cols, s.magic, &col);
        so = row * s.stride + col;
      }
      v[k] = load_stream(reinterpret_cast<const f32x4*>(src + so));
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const uint32_t u = tile.unit0 + k * kThreads + threadIdx.x;
      const uint32_t w0 = cvt_pk_bf16(v[k].x, v[k].y);
      const uint32_t w1 = cvt_pk_bf16(v[k].z, v[k].w);
      if (u <= last) {
        const uint32_t e = u * 4;
        store_stream((u32x2){w0, w1}, reinterpret_cast<u32x2*>(out + e));
        const uint32_t rel = e >> 1;
        acc_w += (uint64_t)w0 + w1;
        acc_rw += (uint64_t)rel * w0 + (uint64_t)(rel + 1) * w1;
      }
    }
  } else {
    // Unaligned segment (a source offset, destination offset or row that is no whole group of 4
    // elements): groups of 4 elements on the destination's 8-byte grid (tile_index.h).
    Group v[kGroups];
#pragma unroll
    for (int k = 0; k < kGroups; ++k) {
      const int32_t e = group_elem(tile.unit0, k, threadIdx.x, lead);
      load_group(src, s, e, v[k]);
    }
#pragma unroll
    for (int k = 0; k < kGroups; ++k) {
      const int32_t e = group_elem(tile.unit0, k, threadIdx.x, lead);
      f32x4 x = v[k].a;
      if (v[k].cut < 4) {
#pragma unroll
        for (int j = 1; j < 4; ++j) x[j] = (uint32_t)j < v[k].cut ? x[j] : v[k].b[j];
      }
      const uint32_t w0 = cvt_pk_bf16(x.x, x.y);
      const uint32_t w1 = cvt_pk_bf16(x.z, x.w);
      if (whole_group(s, e)) {
        store_stream((u32x2){w0, w1}, reinterpret_cast<u32x2*>(out + e));
      } else {
        const uint16_t h[4] = {(uint16_t)w0, (uint16_t)(w0 >> 16), (uint16_t)w1, (uint16_t)(w1 >> 16)};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (e + j >= 0 && (uint32_t)(e + j) < s.units) out[e + j] = h[j];
      }
      // elements outside the segment were loaded as 0 and add nothing to either sum
      const uint32_t rel = (uint32_t)(e + (int32_t)lead) >> 1;
      acc_w += (uint64_t)w0 + w1;
      acc_rw += (uint64_t)rel * w0 + (uint64_t)(rel + 1) * w1;
    }
    uint32_t x;
    if (tail_elem(s, tile.unit0, threadIdx.x, lead, &x)) {
      uint32_t col;
      const uint32_t so = elem_src(s, x, &col);
      const uint32_t bf = cvt_pk_bf16(load_stream(src + so), 0.f) & 0xFFFFu;
      out[x] = (uint16_t)bf;
      const uint32_t q = lead + x;  // element position relative to the first group
      const uint32_t val = bf << ((q & 1) * 16);
      acc_w += val;
      acc_rw += (uint64_t)(q >> 1) * val;
    }
  }
  block_sum2(acc_w, acc_rw, red);
  const uint64_t s2 = (((pos0 - lead) >> 1) + 1) * acc_w + acc_rw;
  if (kOwnSums) {
    if (threadIdx.x < 64) finish_tile_sums(a.sum, g, s.chunk, acc_w, s2);
  } else if (threadIdx.x == 0) {
    add_tile_sums(a.sum, g, s.chunk, acc_w, s2);
  }
}

// One workgroup per tile (grid-stride when the grid is capped).
template <int K, bool kOwnSums>
__global__ __launch_bounds__(kThreads) void stage_kernel(StageArgs args) {
  (void)args;  // read below through the kernarg segment (same bytes)
  const StageArgs& a = *(const StageArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  __shared__ uint64_t red[2][kThreads / 64];
  // The grid holds at most ntiles workgroups: the first tile needs no check, so its arguments load at once.
  // 50 tiny packs replayed from a graph 6.49 us each against 6.58 with the check, 0.5B 568.9 against 570.3.
  uint32_t b = blockIdx.x;
  do {
    const uint32_t t = a.grouped ? xcd_group<kTileGroup>(b, a.ntiles) : xcd_tile(b, a.ntiles);
    stage_tile<K, kOwnSums>(a, a.tile0 + t, red);
    b += a.grid;
  } while (b < a.ntiles);
}

// The path through host memory: packs tiles [tile0, tile0 + ntiles) into pinned host memory (dst)
// and reloads what the previous launch packed.  Bound by the host link, which moves both
// directions at once at about 49 GB/s each way as long as both are kept equally busy: each
// workgroup therefore alternates, K/2 16-byte reload groups per lane (a tile's output bytes)
// in flight across each tile it packs.  Probe, each way: a packing kernel beside a copy engine's
// reload 42.5 GB/s for 64 MiB chunks and 32 for 8 MiB (two event waits across queues per
// chunk); packing and reloading workgroups side by side in one launch 17-46, by their numbers;
// alternating 47.9 and 45.9.  0.5B weights in 64 MiB chunks 30.1 -> 26.7 ms.
struct StageRelayArgs {
  StageArgs s;
  const u32x4* from;  // pinned, 16-byte groups of the previous launch
  u32x4* to;
  uint32_t groups;
};

template <int K>
__global__ __launch_bounds__(kThreads) void stage_relay_kernel(StageRelayArgs args) {
  (void)args;  // read through the kernarg segment (same bytes)
  const StageRelayArgs& a = *(const StageRelayArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  __shared__ uint64_t red[2][kThreads / 64];
  constexpr int R = K / 2;
  const uint32_t reloads = (a.groups + kThreads * R - 1) / (kThreads * R), steps = max(a.s.ntiles, reloads);
  for (uint32_t b = blockIdx.x; b < steps; b += gridDim.x) {
    const uint32_t u0 = b * (kThreads * R) + threadIdx.x;
    u32x4 v[R];
    if (b < reloads) {
#pragma unroll
      for (int k = 0; k < R; ++k) v[k] = load_stream(a.from + min(u0 + k * kThreads, a.groups - 1));
    }
    if (b < a.s.ntiles) stage_tile<K, false>(a.s, a.s.tile0 + b, red);
    if (b < reloads) {
#pragma unroll
      for (int k = 0; k < R; ++k)
        if (u0 + k * kThreads < a.groups) store_stream(v[k], a.to + u0 + k * kThreads);
    }
  }
}

// Chunk sums: for each chunk c in [chunk0, chunk0 + nchunks), out[c - out_chunk0]
// = the sum of the chunk's accumulator slots, which are then set to zero.  Runs
// after the tile kernel on the same stream, so every add has landed.  The sums
// are integer, so the order of the adds does not change the bits.  A lane per
// slot, so every load is in flight at once: one lane per chunk when a chunk has
// one slot (small budgets: up to 10^6 chunks), one wave per chunk up to 64
// slots, one workgroup per chunk beyond; the grid is capped and strides over
// the chunks.
constexpr uint32_t kMaxSumGrid = 1u << 14;
static_assert(kMaxSumSlots <= kThreads, "one lane per accumulator slot");

__global__ __launch_bounds__(kThreads) void chunk_sum_kernel(ChunkSum cs, uint32_t chunk0, uint32_t nchunks) {
  const u64x2 zero = {0, 0};
  if (cs.sub == 1) {
    for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < nchunks; i += gridDim.x * kThreads) {
      const uint32_t c = chunk0 + i;
      u64x2* p = reinterpret_cast<u64x2*>(cs.acc + (uint64_t)(c - cs.chunk_bias) * cs.stride_words);
      const u64x2 v = *p;
      *p = zero;
      *reinterpret_cast<u64x2*>(&cs.out[c - cs.out_chunk0]) = v;
    }
    return;
  }
  if (cs.sub <= 64) {
    const uint32_t lane = threadIdx.x & 63, waves = kThreads / 64;
    // i is the same on every lane of a wave, so the whole wave runs each iteration (DPP sums)
    for (uint32_t i = blockIdx.x * waves + threadIdx.x / 64; i < nchunks; i += gridDim.x * waves) {
      const uint32_t c = chunk0 + i;
      uint64_t a1 = 0, a2 = 0;
      if (lane < cs.sub) {
        const uint64_t slot = (uint64_t)(c - cs.chunk_bias) * cs.sub + lane;
        u64x2* p = reinterpret_cast<u64x2*>(cs.acc + slot * cs.stride_words);
        const u64x2 v = *p;
        *p = zero;
        a1 = v.x;
        a2 = v.y;
      }
      a1 = wave_sum_to_lane63(a1);
      a2 = wave_sum_to_lane63(a2);
      if (lane == 63) *reinterpret_cast<u64x2*>(&cs.out[c - cs.out_chunk0]) = (u64x2){a1, a2};
    }
    return;
  }
  __shared__ uint64_t red[2][kThreads / 64];
  for (uint32_t i = blockIdx.x; i < nchunks; i += gridDim.x) {
    const uint32_t c = chunk0 + i;
    uint64_t a1 = 0, a2 = 0;
    if (threadIdx.x < cs.sub) {
      u64x2* p = reinterpret_cast<u64x2*>(cs.acc + ((uint64_t)(c - cs.chunk_bias) * cs.sub + threadIdx.x) *
                                                       cs.stride_words);
      const u64x2 v = *p;
      *p = zero;
      a1 = v.x;
      a2 = v.y;
    }
    block_sum2(a1, a2, red);
    if (threadIdx.x == 0) *reinterpret_cast<u64x2*>(&cs.out[c - cs.out_chunk0]) = (u64x2){a1, a2};
  }
}

__global__ __launch_bounds__(kThreads) void zero_words_kernel(uint64_t* p, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (uint64_t)gridDim.x * kThreads) p[i] = 0;
}

}  // namespace

hipError_t launch_zero_words(uint64_t* p, uint64_t n, hipStream_t st) {
  if (!n) return hipSuccess;
  const uint32_t grid = (uint32_t)std::min<uint64_t>((n + kThreads - 1) / kThreads, kMaxSumGrid);
  hipLaunchKernelGGL(zero_words_kernel, dim3(grid), dim3(kThreads), 0, st, p, n);
  return hipGetLastError();
}

hipError_t launch_chunk_sums(const ChunkSum& cs, uint32_t chunk0, uint32_t nchunks, hipStream_t st) {
  if (!nchunks) return hipSuccess;
  const uint32_t per = cs.sub == 1 ? kThreads : cs.sub <= 64 ? kThreads / 64 : 1;
  const uint32_t grid = std::min((nchunks + per - 1) / per, kMaxSumGrid);
  hipLaunchKernelGGL(chunk_sum_kernel, dim3(grid), dim3(kThreads), 0, st, cs, chunk0, nchunks);
  return hipGetLastError();
}

namespace {

StageArgs stage_args(const StageLaunch& l) {
  StageArgs args;
  std::memset(&args, 0, sizeof(args));
  args.segs = l.segs;
  args.tiles = l.tiles;
  args.dst = static_cast<uint16_t*>(l.dst);
  args.sum = l.sum;
  args.dst_bias = l.dst_bias;
  args.chunk_elems = l.chunk_elems;
  args.tile0 = l.tile0;
  args.ntiles = l.ntiles;
  args.grouped = l.grouped;
  for (int w = 0; w < l.num_shards; ++w) args.shards[w] = l.shards[w];
  return args;
}

}  // namespace

hipError_t launch_stage_kernel(const StageLaunch& l, hipStream_t st) {
  if (!l.ntiles) return hipSuccess;
  StageArgs args = stage_args(l);
  const uint32_t cap = DR_GRID_CAP > 0 ? (uint32_t)DR_GRID_CAP : kMaxGrid;
  const uint32_t grid = l.ntiles < cap ? l.ntiles : cap;
  args.grid = grid;
  const bool own = l.sum.chunk_tiles != nullptr;
  void (*kernel)(StageArgs) = l.depth == kVecItersLarge
                                  ? (own ? stage_kernel<kVecItersLarge, true> : stage_kernel<kVecItersLarge, false>)
                                  : (own ? stage_kernel<kVecItersSmall, true> : stage_kernel<kVecItersSmall, false>);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), 0, st, args);
  return hipGetLastError();
}

hipError_t launch_stage_relay(const StageLaunch& l, const Reload& r, hipStream_t st) {
  if (!l.ntiles && !r.groups) return hipSuccess;
  StageRelayArgs args;
  args.s = stage_args(l);
  args.from = static_cast<const u32x4*>(r.from);
  args.to = static_cast<u32x4*>(r.to);
  args.groups = r.groups;
  const uint32_t per = kThreads * (l.depth / 2), steps = std::max(l.ntiles, (r.groups + per - 1) / per);
  const uint32_t grid = std::min(steps, std::max(1u, kRelayTileBytes / (16 * per)) * kStageRelayGrid);
  if (l.depth == kVecItersLarge)
    hipLaunchKernelGGL(stage_relay_kernel<kVecItersLarge>, dim3(grid), dim3(kThreads), 0, st, args);
  else
    hipLaunchKernelGGL(stage_relay_kernel<kVecItersSmall>, dim3(grid), dim3(kThreads), 0, st, args);
  return hipGetLastError();
}

}  // namespace dr
