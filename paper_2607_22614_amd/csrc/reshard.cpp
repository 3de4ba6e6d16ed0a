// Host side of the training -> training reshard: argument checks, launches and
// the dr_reshard entry point (kernel in reshard.hip).
#include <hip/hip_runtime.h>

#include "dr_internal.h"
#include "kernels.h"

namespace dr {
namespace {

bool aligned16(const void* p) { return p && (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

int check_reshard_args(const dr_plan* p, const float* const* src_shards, float* const* dst_shards,
                       const dr_checksum* d_cks, const char* what) {
  if (!p) return fail(DR_EINVAL, "%s: null plan", what);
  if (p->kind != kReshard) return fail(DR_EINVAL, "%s: not a reshard plan", what);
  if (!src_shards || !dst_shards) return fail(DR_EINVAL, "%s: null shard array", what);
  for (int w = 0; w < p->layout.train_shards; ++w)
    if (!aligned16(src_shards[w])) return fail(DR_EINVAL, "%s: source shard %d is null or not 16-byte aligned", what, w);
  for (int w = 0; w < p->dst_shards; ++w)
    if (!aligned16(dst_shards[w]))
      return fail(DR_EINVAL, "%s: destination shard %d is null or not 16-byte aligned", what, w);
  if (!aligned16(d_cks)) return fail(DR_EINVAL, "%s: d_cks is null or not 16-byte aligned", what);
  if (!p->d_segs) return fail(DR_EINVAL, "%s: host-only plan has no device tables", what);
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(DR_EHIP, "%s: hipGetDevice: %s", what, hipGetErrorString(e));
  if (dev != p->device) return fail(DR_EINVAL, "%s: plan lives on device %d, current device is %d", what, p->device, dev);
  return DR_OK;
}

ReshardLaunch reshard_launch(const dr_plan* p, const float* const* src, float* const* dst, const ChunkSum& cs) {
  ReshardLaunch l{};
  l.segs = p->d_segs;
  l.tiles = p->tiling[0].d_tiles;
  l.sum = cs;
  l.chunk_elems = p->layout.chunk_bytes / 4;
  l.dst_shard_elems = p->dst_shard_elems;
  l.num_src = p->layout.train_shards;
  l.src = src;
  l.num_dst = p->dst_shards;
  l.dst = dst;
  return l;
}

namespace {

// Reshards that read and write more than this move whole tiles per workgroup, smaller ones half tiles:
// at 43 GB (40.3 GiB) halves are 1-2 % faster, at 50 GB (46.9 GiB) whole tiles 0.5-1 %, at 57 GB 1.5 %
// (the table at the kernel).
constexpr uint64_t kWholeTileBytes = 44ull << 30;

// Tiles [tile0, tile0 + ntiles) of a reshard plan; flat (if not null) receives the destination
// elements from flat_bias on instead of the destination shards.  The tiles cover chunks
// [chunk0, chunk0 + nchunks); the checksum of chunk c goes to cks[c - chunk0].
int launch_reshard(dr_plan* p, uint32_t tile0, uint32_t ntiles, const float* const* src, float* const* dst,
                   float* flat, uint64_t flat_bias, uint32_t chunk0, uint32_t nchunks, dr_checksum* cks,
                   hipStream_t st, const char* what) {
  if (int rc = clear_sums(p, p->tiling[0], chunk0, nchunks, st, what)) return rc;
  ReshardLaunch l = reshard_launch(p, src, dst, chunk_sum(p, p->tiling[0], cks, chunk0));
  l.tile0 = tile0;
  l.ntiles = ntiles;
  l.flat = flat;
  l.flat_bias = flat_bias;
  l.whole_tiles = !flat && 4 * p->info.n_elems + p->info.rollout_bytes > kWholeTileBytes;
  hipError_t e = launch_reshard_kernel(l, st);
  const char* step = "kernel launch";
  if (e == hipSuccess) {
    step = "chunk sum launch";
    e = launch_chunk_sums(l.sum, chunk0, nchunks, st);
  }
  if (e == hipSuccess) return DR_OK;
  mark_sums(p, p->tiling[0]);
  return fail(DR_EHIP, "%s: %s: %s", what, step, hipGetErrorString(e));
}

}  // namespace

// Chunk `chunk` of the destination stream into chunk_dst (bytes [c*B, ...) of the flat
// destination, read from the source shards) and its checksum into *ck.  Arguments checked.
int launch_reshard_chunk(dr_plan* p, uint64_t chunk, const float* const* src, void* chunk_dst, dr_checksum* ck,
                         hipStream_t st, const char* what) {
  const Tiling& tl = p->tiling[0];
  const uint32_t t0 = tl.chunk_tile_begin[chunk], t1 = tl.chunk_tile_begin[chunk + 1];
  const uint64_t ce = p->layout.chunk_bytes / 4;
  return launch_reshard(p, t0, t1 - t0, src, nullptr, static_cast<float*>(chunk_dst), chunk * ce, (uint32_t)chunk, 1,
                        ck, st, what);
}

}  // namespace dr

using namespace dr;

extern "C" int dr_reshard(dr_plan* p, const float* const* src_shards, float* const* dst_shards, dr_checksum* d_cks,
                          void* stream) {
  clear_error();
  if (int rc = check_reshard_args(p, src_shards, dst_shards, d_cks, "dr_reshard")) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  return launch_reshard(p, 0, (uint32_t)p->info.num_tiles, src_shards, dst_shards, nullptr, 0, 0,
                        (uint32_t)p->info.num_chunks, d_cks, st, "dr_reshard");
}
